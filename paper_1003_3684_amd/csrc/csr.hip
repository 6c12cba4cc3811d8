// Edge list -> compressed sparse rows, and the degree histogram.
//
// Entries (src, dst) are packed into one unsigned key (src << db) | dst, with
// db = bits(n - 1) (rounded up to a whole digit when in-degrees are needed),
// and sorted by a least-significant-digit radix sort with 8-bit digits over
// the live key bits.  One histogram pass counts every digit of every pass
// (or, for Kronecker edges generated by the same call, the sampler counts
// them as it writes the ids); each digit pass is then a single "onesweep" kernel: workgroup b takes tile
// b (8,192 keys; with one look-back kernel on the GPU at a time, workgroups
// start in id order, so every tile waited for is already running), ranks its
// keys stably in LDS, publishes its per-digit
// counts and finds the counts of all earlier tiles by decoupled look-back,
// then writes its keys digit run by digit run (coalesced).  One read and one
// write of every key per pass -- the pass is HBM-bound.  The first pass reads
// the edge arrays and packs keys on the fly, so no separate packing pass
// exists.
//
// Without SIMPLE the last digit pass writes the columns itself, marks the
// first sorted position of every row (its row start) and counts repeated
// entries, comparing each key with the one before it in its tile's digit run;
// a small kernel settles the first entry of every run from the run records
// and the look-back counts.  With SIMPLE, one streaming pass after the sort
// does this and drops self-loops and repeats, compacting by a look-back scan.  Rows with no entry are filled by a reverse min-scan over
// the row starts.  The degree histogram counts deg(v) = out + in per vertex
// (the degree distributions of the paper's Results section).  For a directed
// CSR the in-degrees come from the sort itself: once the digit passes over
// the destination field are done the keys are ordered by destination, and the
// next pass marks where each destination's run starts (a column-start array
// filled like the row starts) -- no atomics.
#include <string.h>

#include <algorithm>
#include <mutex>

#include "common.hpp"
#include "kron.hpp"
#include "power.hpp"

namespace sfg {
namespace {

constexpr int kPassThreads = 1024;
constexpr int kPassItems = 8;
constexpr int kPassTile = kPassThreads * kPassItems;  // keys per onesweep tile
// Lists of up to kShortList entries are sorted in shorter tiles: a pass over a
// few tiles takes as long as one tile, and a tile of two keys per thread is ranked
// in a quarter of the steps.  The build in us with 8 and with 2 keys per thread: 52.8 /
// 41.1 for 8,192 entries, 63.9 / 61.2 for 65,536, 77.6 / 76.0 for 262,144, 90.2 /
// 91.2 for 524,288, where the look-back over four times the tiles costs what the
// ranking saves.  The short tiles' look-back words are 32-bit, and those of more
// than kShortTiles tiles would not fit what a plan reserves for the long tiles, so
// such a list takes kMidItems keys per thread (100,000 directed entries over 3,000
// vertices: 67.5 with 8, 57.4 with 3, 58.7 with 2).  A workspace that grew for the
// short tiles would be too small for a list of kShortList entries when it was
// sized for a longer one.
constexpr int kShortItems = 2, kMidItems = 3;
constexpr uint64_t kShortTiles = 30;
constexpr uint64_t kShortList = 131072;
constexpr uint64_t kSpareTiles = 7;  // long tiles' look-back words beyond a plan's own
constexpr int kPassWaves = kPassThreads / 64;
constexpr int kRadix = 256;
constexpr int kLookWindow = 2;  // predecessors read per lane and look-back round trip
constexpr int kLanesPerDigit = kPassThreads / kRadix;  // look-back lanes per digit

constexpr int kPlainThreads = 256;

// Threads of a finish workgroup and keys of a thread.  Every tile's look-back
// reads the words of the tiles in flight before it, past the caches, so the
// words read are the tiles times the tiles in flight and a larger tile saves
// both ways, as long as two workgroups fit a CU.  csr_finish in us for 4.8e7
// 8-byte keys (SIMPLE) at 256 threads x 16 keys / 256 x 32 / 512 x 12 / 512 x 16 / 512 x
// 24 / 1024 x 8 / 1024 x 12: 227 / 200 / 213 / 200 / 201 / 205 / 233.  XOR of 2.1e8 and
// 1e8 entries at 256 x 16 / 512 x 8 / 512 x 12 / 512 x 16: 2,562 / 2,469 / 2,605 /
// 2,398.
constexpr int kFinThreads = 512, kFinItems = 16;
constexpr int kFinTile = kFinThreads * kFinItems;
constexpr int kXorThreads = 512, kXorItems = 16;
// Fewer entries make shorter tiles: a thread's entries are walked one after the
// other, and over a power of sparse rows most of them are looked up from the top, so
// that a tile is a long chain which a few tiles do not hide.  The whole graph in us
// with 16 / 8 / 4 entries per thread: 8,192 entries in rows of one, with 50,000 random pairs, 157 /
// 131 / 116; 248,832 with as many, rows of 12^5 / 8^5, 129 / 114 / 106; 1,771,561 with 50,000
// 97 / 91 / 95, with 7,086,244 314 / 300 / 323; 19,487,171 alone 112 / 121 / 181, with as many random
// pairs 922 / 919 / 1,043.
constexpr int kXorMidItems = 8, kXorShortItems = 4;
constexpr uint64_t kXorShort = 1 << 20, kXorMid = 1 << 24;  // entries, at most
constexpr int xor_items(uint64_t entries) {
    return entries <= kXorShort ? kXorShortItems : entries <= kXorMid ? kXorMidItems : kXorItems;
}
constexpr uint64_t xor_tiles(uint64_t entries, int items) { return (entries + kXorThreads * items - 1) / (kXorThreads * items); }

constexpr int kScanChunk = 4096;  // vertices per chunk of the row fill scan
constexpr int kPrepThreads = 1024;
constexpr int kPrepUnroll = 4;    // keys per thread in flight in the histogram pass
// Interleaved copies of each LDS histogram.  Lanes of a wave that count the same
// digit in the same copy wait for each other, and in a list that comes sorted
// by source (PBA) whole waves share the high digits of it: csr_prepare in us of
// 6.7e8 such edges / 2.4e7 unordered ones with 4 copies in four workgroups of
// 256 threads per CU 4,725 / 96, with 8 in two of 1,024 2,657 / 97, with 16 in one
// (128 KB of LDS) 1,701 (3.2 TB/s) / 96 (4 TB/s).  Counting a digit that all lanes
// share with one add cost more instructions than it saved (2,747 -> 3,460).
constexpr int kPrepCopies = 16;
constexpr int kPrepBlocksPerCu = 1;
constexpr int kPrepMinEdges = 4096;  // edges a workgroup of it has at least

constexpr uint64_t kNoRow = ~0ull;

// Look-back status word: pass tag in the top 6 bits, flag in the next 2, then
// the count: 56 bits, or 24 in a 32-bit word.
constexpr uint64_t kFlagAgg = 1, kFlagIncl = 2;
static_assert(kShortList < (1u << 24), "a short list's counts fit 24 bits");
// (of the passes in tiles of ITEMS keys per thread)
template <int ITEMS> using StatusWord = typename std::conditional<(ITEMS < kPassItems), uint32_t, uint64_t>::type;
template <typename WordT> constexpr int kCountBits = sizeof(WordT) * 8 - 8;
template <typename WordT = uint64_t> __device__ __forceinline__ WordT status_word(uint32_t tag, uint64_t flag, uint64_t v) {
    return ((WordT)tag << (kCountBits<WordT> + 2)) | ((WordT)flag << kCountBits<WordT>) | (WordT)v;
}
template <typename WordT> __device__ __forceinline__ uint32_t status_tag(WordT v) { return (uint32_t)(v >> (kCountBits<WordT> + 2)); }
template <typename WordT> __device__ __forceinline__ uint64_t status_flag(WordT v) { return (v >> kCountBits<WordT>) & 3; }
template <typename WordT> __device__ __forceinline__ uint64_t status_count(WordT v) {
    return v & (((WordT)1 << kCountBits<WordT>) - 1);
}

__device__ __forceinline__ uint32_t count_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// Sum-scan over the first 256 threads of a block (4 waves): returns the
// exclusive prefix of v and writes the total to *total.  All threads of the
// block must call it.
__device__ uint64_t block_exclusive_scan_256(uint64_t v, uint64_t *s_tmp /*[4]*/, uint64_t *total) {
    const int tid = threadIdx.x;
    const uint32_t lane = tid & 63;
    const int w = tid >> 6;
    uint64_t x = tid < 256 ? v : 0;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint64_t y = __shfl_up(x, off, 64);
        if (lane >= (uint32_t)off) x += y;
    }
    if (tid < 256 && lane == 63) s_tmp[w] = x;
    __syncthreads();
    uint64_t base = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (i < w) base += s_tmp[i];
        tot += s_tmp[i];
    }
    __syncthreads();
    *total = tot;
    return base + x - (tid < 256 ? v : 0);
}

// Exclusive prefix of v over the THREADS threads of a block, *total their sum.
// All threads of the block must call it; s_tmp may be used again after.
template <int THREADS> __device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *s_tmp /*[THREADS / 64]*/, uint32_t *total) {
    const uint32_t lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(x, off, 64);
        if (lane >= (uint32_t)off) x += y;
    }
    if (lane == 63) s_tmp[w] = x;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < THREADS / 64; ++i) {
        if (i < w) base += s_tmp[i];
        tot += s_tmp[i];
    }
    __syncthreads();
    *total = tot;
    return base + x - v;
}

// (u << wb) | v, with v cut to wb bits: an id outside [0, 2^wb) then changes
// only its own field, so the key digits always agree with what the histogram
// pass counts (whichever way it counts them) and no pass writes out of range.
template <typename IdT, typename KeyT> __device__ __forceinline__ KeyT pack(IdT u, IdT v, int wb) {
    using U = typename std::conditional<sizeof(IdT) == 4, uint32_t, uint64_t>::type;
    return ((KeyT)(U)u << wb) | ((KeyT)(U)v & (((KeyT)1 << wb) - 1));
}

// Key number idx of the (optionally symmetrized) entry sequence.
template <typename IdT, typename KeyT, bool SYM>
__device__ __forceinline__ KeyT entry_key(const IdT *src, const IdT *dst, uint64_t E, uint64_t idx, int wb) {
    if (!SYM || idx < E) return pack<IdT, KeyT>(src[idx], dst[idx], wb);
    const uint64_t j = idx - E;
    return pack<IdT, KeyT>(dst[j], src[j], wb);
}

// --------------------------------------------------------------------------- prepare
struct PrepArgs {
    uint64_t E, N;
    const void *src, *dst;
    uint64_t *ghist;   // [passes][256]
    int wb, passes;    // wb: width of the destination field
    int dbytes;        // SYM with a whole-byte destination field: its bytes, else 0
};

// One count of every digit of k (all lanes of their copy of the histograms).
template <typename KeyT> __device__ __forceinline__ void count_digits(uint32_t *s_h, KeyT k, int passes, uint32_t copy) {
#pragma unroll
    for (int p = 0; p < (int)sizeof(KeyT); ++p)
        if (p < passes) atomicAdd(&s_h[(p * kRadix + (uint32_t)((k >> (8 * p)) & 255)) * kPrepCopies + copy], 1u);
}

template <typename IdT, typename KeyT, bool SYM>
__global__ __launch_bounds__(kPrepThreads) void csr_prepare(PrepArgs a) {
    // kPrepCopies interleaved copies of every histogram, lane l counting in
    // copy l mod kPrepCopies: skewed digits (one value drawn by many lanes of
    // a wave) would otherwise serialise the LDS atomics on one address.
    __shared__ uint32_t s_h[8 * kRadix * kPrepCopies];
    const int rows = SYM && a.dbytes ? a.dbytes : a.passes;
    for (int i = threadIdx.x; i < rows * kRadix * kPrepCopies; i += kPrepThreads) s_h[i] = 0;
    __syncthreads();
    const uint32_t copy = threadIdx.x % kPrepCopies;
    const IdT *src = static_cast<const IdT *>(a.src), *dst = static_cast<const IdT *>(a.dst);
    // kPrepUnroll keys per thread are loaded before any is counted, so that
    // enough loads are in flight to cover the memory latency.
    // Every edge is read once; with SYM its reversed entry is counted too.
    const uint64_t stride = (uint64_t)gridDim.x * kPrepThreads * kPrepUnroll;
    for (uint64_t i0 = (uint64_t)blockIdx.x * kPrepThreads * kPrepUnroll + threadIdx.x; i0 < a.E; i0 += stride) {
        IdT su[kPrepUnroll], du[kPrepUnroll];
#pragma unroll
        for (int u = 0; u < kPrepUnroll; ++u) {
            const uint64_t i = min(i0 + (uint64_t)u * kPrepThreads, a.E - 1);
            su[u] = src[i];
            du[u] = dst[i];
        }
#pragma unroll
        for (int u = 0; u < kPrepUnroll; ++u) {
            const uint64_t i = i0 + (uint64_t)u * kPrepThreads;
            if (i >= a.E) break;
            if (SYM && a.dbytes) {
                // Key byte p of (u, v) and of (v, u) together is byte p mod
                // dbytes of u plus that of v: one count per byte of each end.
                using U = typename std::conditional<sizeof(IdT) == 4, uint32_t, uint64_t>::type;
                count_digits<U>(s_h, (U)su[u], a.dbytes, copy);
                count_digits<U>(s_h, (U)du[u], a.dbytes, copy);
                continue;
            }
            count_digits<KeyT>(s_h, pack<IdT, KeyT>(su[u], du[u], a.wb), a.passes, copy);
            if (SYM) count_digits<KeyT>(s_h, pack<IdT, KeyT>(du[u], su[u], a.wb), a.passes, copy);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < a.passes * kRadix; i += kPrepThreads) {
        // (with dbytes, pass p's histogram is the byte histogram p mod dbytes)
        const int row = (SYM && a.dbytes) ? (i / kRadix) % a.dbytes * kRadix + i % kRadix : i;
        uint32_t t = 0;
#pragma unroll
        for (int c = 0; c < kPrepCopies; ++c) t += s_h[row * kPrepCopies + c];
        if (t) atomicAdd((unsigned long long *)&a.ghist[i], (unsigned long long)t);
    }
}

// --------------------------------------------------------------------------- onesweep pass

struct PassArgs {
    uint64_t E, N;
    const void *src, *dst;  // first pass only
    const void *in;         // later passes
    void *out;
    void *status;           // [tiles][256] look-back words (StatusWord<ITEMS>)
    uint64_t *gbase;        // [256] bucket bases of a FINAL pass, left for csr_run_starts
    const uint64_t *ghist;  // [256] of this pass: digits no entry has skip the look-back
    uint32_t *err;
    uint64_t *csc;          // column starts (BOUND passes only)
    uint8_t *cmark;         // 1 where a column start was written (BOUND passes only)
    int wb, shift;          // wb: width of the destination field
    uint32_t tag;
    uint64_t nv;            // vertices (BOUND passes write column starts below it)
    // FINAL pass only: the CSR outputs and the run records (see radix_pass).
    void *col;
    uint64_t *rp;
    uint8_t *mark;
    void *run_first, *run_last;  // [tiles][256] keys
    uint32_t *tile_dups;         // [tiles]
    // FINAL pass over packed ids: the columns are written unpacked, group j
    // of dec_bits bits taken from dec[byte j of the packed id].
    const uint32_t *dec;
    int dec_groups, dec_bits;
};

// The id of a packed id (see ByteCount in kron.hpp).
template <typename KeyT>
__device__ __forceinline__ uint64_t unpack_id(KeyT packed, const uint32_t *dec, int groups, int bits) {
    uint64_t id = 0;
    for (int j = groups - 1; j >= 0; --j) id = (id << bits) | dec[(uint32_t)(packed >> (8 * j)) & 255u];
    return id;
}

// BOUND: the input keys are ordered by destination; mark the first position
// of every destination run in csc.
// FINAL (the last pass of a CSR without SIMPLE): the output order is the
// sorted order, so the pass writes the columns instead of the keys, and marks
// row starts and counts repeated entries wherever the previous sorted entry is
// the previous key of the same digit run in this tile.  The first entry of a
// run follows an entry of another tile (or of another digit's bucket); the
// run's first and last keys go to the run records, and csr_run_starts
// settles those entries once every tile is done.
template <typename IdT, typename KeyT, bool SYM, bool FIRST, bool BOUND, bool FINAL, int ITEMS>
__global__ __launch_bounds__(kPassThreads, ITEMS < kPassItems ? 4 : BOUND ? 6 : 8) void radix_pass(PassArgs a) {
    constexpr int kItems = ITEMS, kTile = kPassThreads * kItems;
    // s_keys holds the tile's keys in digit order after ranking; during the
    // ranking its first 32 KB serve as the per-wave lane-match tables.
    constexpr size_t kMatchBytes = sizeof(uint64_t) * kPassWaves * kRadix;
    __shared__ __align__(16) KeyT s_keys[kTile * sizeof(KeyT) > kMatchBytes ? kTile : kMatchBytes / sizeof(KeyT)];
    // 16-bit per-wave digit counters (8 KB); with the 64 KB key tile the block takes about 77 KB of LDS
    // (8-byte keys): two workgroups per CU.
    __shared__ uint16_t s_cnt[kPassWaves][kRadix];
    __shared__ uint16_t s_off[kRadix];
    __shared__ uint16_t s_tot[kRadix];
    __shared__ uint64_t s_gpos[kRadix];
    __shared__ uint64_t s_tmp[4];
    // FINAL over packed ids: the byte -> digit-group table, read once per key.
    __shared__ uint32_t s_dec[FINAL ? kRadix : 1];
    static_assert(kPassThreads % kRadix == 0 && 64 % kLanesPerDigit == 0, "look-back lane groups");
    uint64_t *s_match = reinterpret_cast<uint64_t *>(s_keys) + 0;  // [kPassWaves][256]

    using WordT = StatusWord<ITEMS>;
    WordT *status = static_cast<WordT *>(a.status);
    const int tid = threadIdx.x;
    const uint32_t lane = tid & 63;
    const int w = tid >> 6;
    // Tile = workgroup id.  While this is the only look-back kernel on the
    // GPU, workgroups start in id order (each XCD takes its share of the ids
    // in order), so every tile this one waits for started earlier and is
    // running or done: the smallest unfinished tile never waits.  Two
    // look-back kernels at once could each hold the XCD space that the
    // other's smallest unfinished tile needs, so the library never runs two
    // (the ensemble keeps one stream) and callers must not overlap sorting
    // calls on one device.  (A ticket counter would serialise the tiles on
    // one device-coherent atomic.)
    const uint64_t tile = blockIdx.x;
    const uint64_t tile_base = tile * kTile;
    const uint64_t wbase = tile_base + (uint64_t)w * 64 * kItems;
    const bool full = tile_base + kTile <= a.N;

    // The keys' loads go out first; the LDS counters are cleared while they
    // travel.
    KeyT k[kItems];
    uint32_t d[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const uint64_t idx = wbase + (uint64_t)i * 64 + lane;
        const bool valid = full || idx < a.N;
        if (FIRST)
            k[i] = valid ? entry_key<IdT, KeyT, SYM>(static_cast<const IdT *>(a.src), static_cast<const IdT *>(a.dst),
                                                      a.E, idx, a.wb)
                         : (KeyT)0;
        else
            k[i] = valid ? static_cast<const KeyT *>(a.in)[idx] : (KeyT)0;
    }
    const bool used = a.ghist[(uint32_t)tid / kLanesPerDigit] != 0;
    for (int i = tid; i < kPassWaves * kRadix; i += kPassThreads) {
        (&s_cnt[0][0])[i] = 0;
        s_match[i] = 0;
    }
    if (FINAL && a.dec && tid < kRadix) s_dec[tid] = a.dec[tid];
    __syncthreads();
    // The buckets' bases enter the prefixes through tile 0, whose published
    // counts start from them (a scan of the digit counts that no other tile
    // needs to do, and no launch of its own).
    if (tile == 0) {
        uint64_t entries;
        const uint64_t base = block_exclusive_scan_256(tid < kRadix ? a.ghist[tid] : 0, s_tmp, &entries);
        if (tid < kRadix) {
            s_gpos[tid] = base;
            if (FINAL) a.gbase[tid] = base;
        }
    }
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const uint64_t idx = wbase + (uint64_t)i * 64 + lane;
        d[i] = (full || idx < a.N) ? (uint32_t)(k[i] >> a.shift) & 255u : (uint32_t)kRadix;
    }

    if (BOUND) {
        // The key before position idx: the previous lane of the same item,
        // lane 63 of the previous item, or (first key of the wave) memory.
        const KeyT mask = ((KeyT)1 << a.wb) - 1;
        const KeyT *in = static_cast<const KeyT *>(a.in);
        KeyT carry = (wbase > 0 && wbase <= a.N) ? in[wbase - 1] : (KeyT)0;
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
            const uint64_t idx = wbase + (uint64_t)i * 64 + lane;
            KeyT prev = __shfl_up(k[i], 1, 64);
            if (lane == 0) prev = carry;
            carry = __shfl(k[i], 63, 64);
            // (ids at or above n are not vertices: never written, never a fault)
            if (idx < a.N && (idx == 0 || (k[i] & mask) != (prev & mask)) && (uint64_t)(k[i] & mask) < a.nv) {
                a.csc[(uint64_t)(k[i] & mask)] = idx;
                a.cmark[(uint64_t)(k[i] & mask)] = 1;
            }
        }
    }

    // Stable rank inside the wave.  For each group of 64 keys every lane ORs
    // its lane bit into the wave's match slot of its digit; reading the slot
    // back gives the lanes sharing the digit (OR is order-free, so the mask
    // is exact).  Lanes below this one in the mask come first; the lowest
    // lane of each digit advances the wave's counter and clears the slot.
    // LDS operations of one wave complete in program order.
    uint32_t r[kItems];
    uint64_t *match = s_match + w * kRadix;
    uint16_t *wcnt = s_cnt[w];
    const uint64_t my_bit = 1ull << lane;
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const uint32_t di = d[i];
        const bool valid = di < kRadix;
        const uint32_t slot = valid ? di : 0;
        if (valid) atomicOr(reinterpret_cast<unsigned long long *>(&match[slot]), (unsigned long long)my_bit);
        __builtin_amdgcn_wave_barrier();
        const uint64_t peers = valid ? match[slot] : 0ull;
        const uint32_t below = count_below(peers);
        const uint32_t old = wcnt[slot];
        r[i] = old + below;
        __builtin_amdgcn_wave_barrier();
        if (valid && below == 0) {
            wcnt[slot] = (uint16_t)(old + (uint32_t)__popcll(peers));
            match[slot] = 0;
        }
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();

    // Per digit: prefix over the waves and the tile's count.
    uint32_t cnt = 0;
    if (tid < kRadix) {
        uint32_t acc = 0;
#pragma unroll
        for (int wv = 0; wv < kPassWaves; ++wv) {
            const uint32_t c = s_cnt[wv][tid];
            s_cnt[wv][tid] = (uint16_t)acc;
            acc += c;
        }
        cnt = acc;
        s_tot[tid] = (uint16_t)acc;
    }
    __syncthreads();

    // Decoupled look-back with kLanesPerDigit consecutive lanes per digit:
    // lane q of digit d's group reads kLookWindow predecessors, so one round
    // trip covers kLanesPerDigit kLookWindow earlier tiles.  Lane 0 of the
    // group publishes: the tile's own count first, its inclusive prefix once
    // known.
    // A digit that no entry of the pass has (known from the histogram pass)
    // has a zero prefix everywhere: its lanes neither publish nor walk.  Key
    // ranges that leave digit values unused (ids below a power of the radix,
    // generators with zero cells) save that part of the status traffic.
    const uint32_t dg = (uint32_t)tid / kLanesPerDigit, part = (uint32_t)tid % kLanesPerDigit;
    const uint64_t my_cnt = s_tot[dg];
    if (part == 0 && used)
        store_agent(status + tile * kRadix + dg, tile == 0 ? status_word<WordT>(a.tag, kFlagIncl, s_gpos[dg] + my_cnt)
                                                           : status_word<WordT>(a.tag, kFlagAgg, my_cnt));
    const bool walk = tile > 0 && used;

    uint64_t tot;
    const uint64_t ex = block_exclusive_scan_256(cnt, s_tmp, &tot);
    if (tid < kRadix) s_off[tid] = (uint16_t)ex;
    __syncthreads();

    // Scatter into LDS in digit order (the local order needs no global
    // offsets, and the keys leave the registers before the look-back).
#pragma unroll
    for (int i = 0; i < kItems; ++i)
        if (d[i] < kRadix) s_keys[s_off[d[i]] + s_cnt[w][d[i]] + r[i]] = k[i];

    uint64_t prefix = tile == 0 && part == 0 ? s_gpos[dg] : 0;
    if (walk) {
        uint64_t j = tile;  // tiles below j are still to be examined
        for (;;) {
            // This lane's predecessors: j - 1 - (part kLookWindow + i).  One
            // beyond tile 0 reads as an inclusive zero, which ends the walk.
            WordT v[kLookWindow];
#pragma unroll
            for (int i = 0; i < kLookWindow; ++i) {
                const uint64_t back = (uint64_t)part * kLookWindow + i;
                v[i] = j > back ? load_agent(status + (j - 1 - back) * kRadix + dg)
                                : status_word<WordT>(a.tag, kFlagIncl, 0);
            }
            uint64_t sum = 0;
            bool found = false;
#pragma unroll
            for (int i = 0; i < kLookWindow; ++i) {
                if (found) break;
                const uint64_t back = (uint64_t)part * kLookWindow + i;
                uint32_t spins = 0;
                while (status_tag(v[i]) != a.tag) {
                    if (++spins > kSpinLimit || ((spins & 1023) == 0 && load_agent(a.err) != 0)) {
                        raise_device_error(a.err, DEVERR_LOOKBACK);
                        v[i] = status_word<WordT>(a.tag, kFlagIncl, 0);
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                    v[i] = load_agent(status + (j - 1 - back) * kRadix + dg);
                }
                sum += status_count(v[i]);
                found = status_flag(v[i]) == kFlagIncl;
            }
            // Combine the group, nearest predecessors first.
            const int lead = (int)(lane & ~(uint32_t)(kLanesPerDigit - 1));
            bool done = false;
#pragma unroll
            for (int q = 0; q < kLanesPerDigit; ++q) {
                const uint64_t sq = __shfl(sum, lead + q, 64);
                const int fq = __shfl((int)found, lead + q, 64);
                if (!done) {
                    prefix += sq;
                    done = fq != 0;
                }
            }
            if (done) break;
            j -= (uint64_t)kLanesPerDigit * kLookWindow;  // else a sentinel had ended the walk
        }
        if (part == 0) store_agent(status + tile * kRadix + dg, status_word<WordT>(a.tag, kFlagIncl, prefix + my_cnt));
    }
    if (part == 0) s_gpos[dg] = prefix;
    __syncthreads();
    if (tid < kRadix) s_gpos[tid] -= ex;
    __syncthreads();

    // Write the digit runs out, coalesced.
    const uint64_t rem = a.N - tile_base;
    const uint32_t nvalid = rem < (uint64_t)kTile ? (uint32_t)rem : (uint32_t)kTile;
    if (FINAL) {
        IdT *col = static_cast<IdT *>(a.col);
        KeyT *rfirst = static_cast<KeyT *>(a.run_first) + tile * kRadix;
        KeyT *rlast = static_cast<KeyT *>(a.run_last) + tile * kRadix;
        const KeyT mask = ((KeyT)1 << a.wb) - 1;
        uint32_t ndup = 0;
        for (uint32_t p = tid; p < nvalid; p += kPassThreads) {
            const KeyT key = s_keys[p];
            const uint32_t dd = (uint32_t)(key >> a.shift) & 255u;
            const uint64_t pos = s_gpos[dd] + p;
            const KeyT cv = key & mask;
            __builtin_nontemporal_store(a.dec ? (IdT)unpack_id(cv, s_dec, a.dec_groups, a.dec_bits) : (IdT)cv,
                                        &col[pos]);
            const KeyT prev = p > 0 ? s_keys[p - 1] : (KeyT)0;
            const bool starts = p == 0 || ((uint32_t)(prev >> a.shift) & 255u) != dd;
            const bool ends = p + 1 == nvalid || ((uint32_t)(s_keys[p + 1] >> a.shift) & 255u) != dd;
            if (starts) {
                rfirst[dd] = key;
            } else {
                // (ids at or above n are not vertices: never written, never a fault)
                const uint64_t row = (uint64_t)(key >> a.wb);
                if (row != (uint64_t)(prev >> a.wb) && row < a.nv) {
                    a.rp[row] = pos;
                    a.mark[row] = 1;
                }
                ndup += key == prev ? 1u : 0u;
            }
            if (ends) rlast[dd] = key;
        }
        for (int off = 32; off > 0; off >>= 1) ndup += __shfl_xor(ndup, off, 64);
        __syncthreads();  // s_tmp is free again
        uint32_t *s_dup = reinterpret_cast<uint32_t *>(s_tmp);
        if (tid == 0) *s_dup = 0;
        __syncthreads();
        if (lane == 0 && ndup) atomicAdd(s_dup, ndup);
        __syncthreads();
        if (tid == 0) a.tile_dups[tile] = *s_dup;
        return;
    }
    KeyT *out = static_cast<KeyT *>(a.out);
    for (uint32_t p = tid; p < nvalid; p += kPassThreads) {
        const KeyT key = s_keys[p];
        const uint32_t dd = (uint32_t)(key >> a.shift) & 255u;
        // An ordinary (write-back) store: the lines where two tiles' runs of a
        // digit meet are merged in L2 when both halves get there, and the pass
        // times stay the same whichever of the two key buffers the pass
        // writes (streaming stores made one of them about 7% slower).
        out[s_gpos[dd] + p] = key;
    }
}

// --------------------------------------------------------------------------- run starts
// After a FINAL pass: the entries that open a digit run of a tile.  The
// pass's look-back words now hold, for every digit d an entry has and every
// tile t, incl(t, d): the bucket base of d plus the count of digit-d entries in
// tiles <= t, so tile t's run of d starts at incl(t - 1, d).  Its predecessor
// in sorted order is the last entry of the nearest earlier tile with a run of
// d (the first tile whose incl reaches incl(t - 1, d)), or, for the first run
// of d, the last entry of the previous digit that entries have.
struct RunArgs {
    uint64_t tiles, n;
    const void *status;      // [tiles][256] of the FINAL pass
    const uint64_t *gbase;   // [256] bucket bases of that pass
    const uint64_t *ghist;   // [256] digit counts of that pass
    const void *run_first, *run_last;
    const uint32_t *tile_dups;
    uint64_t *rp;
    uint64_t entries;        // rp[n]
    uint8_t *mark;
    uint64_t *dups;
    uint32_t *err;
    int wb;
    uint32_t tag;
    int run_tiles;  // tiles per workgroup, a multiple of kRunBatch
};

// Tiles per workgroup of csr_run_starts: 16, whose counts then roll along,
// where that gives every CU a workgroup, else 4 (the passes' tiles are walked
// one memory latency after the other: 16.4 us for 64 tiles, 9.7 with 4 per workgroup).
constexpr int kRunTiles = 16;

// Inclusive count of a look-back word (0 and a device error when the word is
// not the FINAL pass's inclusive count).
template <typename WordT> __device__ __forceinline__ uint64_t incl_value(const RunArgs &a, WordT v) {
    if (status_tag(v) != a.tag || status_flag(v) != kFlagIncl) {
        raise_device_error(a.err, DEVERR_LOOKBACK);
        return 0;
    }
    return status_count(v);
}

// The FINAL pass has ended, so its look-back words are read with ordinary
// (cacheable) loads.
template <typename WordT> __device__ __forceinline__ uint64_t incl_of(const RunArgs &a, uint64_t t, uint32_t d) {
    return incl_value(a, static_cast<const WordT *>(a.status)[t * kRadix + d]);
}

// Smallest tile x in [lo, hi] with incl(x, d) >= target (incl(hi, d) >= target).
template <typename WordT>
__device__ uint64_t first_tile_reaching(const RunArgs &a, uint32_t d, uint64_t lo, uint64_t hi, uint64_t target) {
    while (lo < hi) {
        const uint64_t mid = lo + (hi - lo) / 2;
        if (incl_of<WordT>(a, mid, d) >= target)
            hi = mid;
        else
            lo = mid + 1;
    }
    return lo;
}

// A workgroup takes run_tiles consecutive tiles, thread d digit d; the
// inclusive counts of the two tiles before the current one roll along.
// The loads of kRunBatch tiles -- look-back word, first key, and the last
// key of the tile before (the usual predecessor) -- go out together.
constexpr int kRunBatch = 4;

template <typename KeyT, typename WordT>
__global__ __launch_bounds__(kRadix) void csr_run_starts(RunArgs a) {
    const WordT *status = static_cast<const WordT *>(a.status);
    __shared__ uint32_t s_dup;
    const uint32_t d = threadIdx.x;
    const bool used = a.ghist[d] != 0;
    const KeyT *first = static_cast<const KeyT *>(a.run_first);
    const KeyT *last = static_cast<const KeyT *>(a.run_last);
    if (d == 0) s_dup = 0;
    if (d == 0 && blockIdx.x == 0) a.rp[a.n] = a.entries;
    __syncthreads();
    uint32_t ndup = 0;
    const uint64_t t0 = (uint64_t)blockIdx.x * a.run_tiles;
    // incl(t - 2, d) and incl(t - 1, d) of the current tile t (the base before tile 0)
    const uint64_t base = a.gbase[d];
    uint64_t c2 = (used && t0 >= 2) ? incl_of<WordT>(a, t0 - 2, d) : base;
    uint64_t c1 = (used && t0 >= 1) ? incl_of<WordT>(a, t0 - 1, d) : base;
    for (int i0 = 0; i0 < a.run_tiles; i0 += kRunBatch) {
        WordT raw[kRunBatch];
        KeyT fk[kRunBatch], lk[kRunBatch];
#pragma unroll
        for (int u = 0; u < kRunBatch; ++u) {
            const uint64_t t = t0 + i0 + u;
            const bool ok = used && t < a.tiles;
            raw[u] = ok ? status[t * kRadix + d] : 0;
            fk[u] = ok ? first[t * kRadix + d] : (KeyT)0;
            lk[u] = (ok && t >= 1) ? last[(t - 1) * kRadix + d] : (KeyT)0;
        }
#pragma unroll
        for (int u = 0; u < kRunBatch; ++u) {
            const uint64_t t = t0 + i0 + u;
            if (t >= a.tiles) break;
            if (d == 0) ndup += a.tile_dups[t];
            if (!used) continue;
            const uint64_t before = c1, before2 = c2;
            const uint64_t cur = incl_value(a, raw[u]);
            c2 = c1;
            c1 = cur;
            if (cur == before) continue;  // no run of d in tile t
            const KeyT f = fk[u];
            bool has = false;
            KeyT pred = 0;
            if (before > base) {
                // the nearest earlier tile with a run of d: usually t - 1
                if (t < 2 || before2 < before) {
                    pred = lk[u];
                } else {
                    const uint64_t tp = first_tile_reaching<WordT>(a, d, 0, t - 2, before);
                    pred = last[tp * kRadix + d];
                }
                has = true;
            } else {
                int dp = (int)d - 1;
                while (dp >= 0 && a.ghist[dp] == 0) --dp;
                if (dp >= 0) {
                    const uint64_t tp = first_tile_reaching<WordT>(a, (uint32_t)dp, 0, a.tiles - 1, a.gbase[dp] + a.ghist[dp]);
                    pred = last[tp * kRadix + dp];
                    has = true;
                }
            }
            const uint64_t pos = before;
            const uint64_t row = (uint64_t)(f >> a.wb);
            if ((!has || row != (uint64_t)(pred >> a.wb)) && row < a.n) {
                a.rp[row] = pos;
                a.mark[row] = 1;
            }
            ndup += (has && f == pred) ? 1u : 0u;
        }
    }
    if (!a.dups) return;
    for (int off = 32; off > 0; off >>= 1) ndup += __shfl_xor(ndup, off, 64);
    if ((d & 63) == 0 && ndup) atomicAdd(&s_dup, ndup);
    __syncthreads();
    if (d == 0 && s_dup) atomicAdd((unsigned long long *)a.dups, (unsigned long long)s_dup);
}

// --------------------------------------------------------------------------- finish
struct FinArgs {
    uint64_t N, n;
    const void *keys;
    void *col;
    uint64_t *rp;       // row starts in output (compacted) positions, written where a row starts
    uint64_t *rp_raw;   // row starts in sorted positions, or null
    uint8_t *mark;      // 1 where a row start was written (shared by rp and rp_raw)
    uint64_t *dups;     // [1] accumulated, or null
    uint64_t *status;   // [tiles] look-back words (SIMPLE)
    uint32_t *err;
    int wb;
    // XOR: `keys` are the random graph's `random` sorted pairs; N counts them
    // and the power's entries together.  split[t]: how many of the random pairs
    // come before the first position of tile t.
    uint64_t random;
    const uint64_t *split;
};

__device__ __forceinline__ int fin_slot(int i) { return i + (i >> 4); }

// Non-SIMPLE finish: one streaming pass with no LDS.  Thread t of a block
// owns positions base + j*256 + t; the key before position idx comes from the
// previous lane (or, for lane 0, from memory).
template <typename IdT, typename KeyT>
__global__ __launch_bounds__(kPlainThreads) void csr_finish_plain(FinArgs a) {
    __shared__ uint32_t s_dups[kPlainThreads / 64];
    const int tid = threadIdx.x;
    const uint32_t lane = tid & 63;
    const KeyT *K = static_cast<const KeyT *>(a.keys);
    IdT *col = static_cast<IdT *>(a.col);
    const KeyT mask = ((KeyT)1 << a.wb) - 1;
    uint32_t ndup = 0;
    const uint64_t stride = (uint64_t)gridDim.x * kPlainThreads;
    for (uint64_t idx = (uint64_t)blockIdx.x * kPlainThreads + tid; idx - lane < a.N; idx += stride) {
        const bool valid = idx < a.N;
        const KeyT key = valid ? K[idx] : (KeyT)0;
        KeyT prev = __shfl_up(key, 1, 64);
        if (lane == 0 && idx > 0 && valid) prev = K[idx - 1];
        if (valid) {
            __builtin_nontemporal_store((IdT)(key & mask), &col[idx]);  // streaming output
            const uint64_t row = (uint64_t)(key >> a.wb);
            if ((idx == 0 || row != (uint64_t)(prev >> a.wb)) && row < a.n) {
                a.rp[row] = idx;
                if (a.rp_raw) a.rp_raw[row] = idx;
                a.mark[row] = 1;
            }
            ndup += (idx > 0 && key == prev) ? 1u : 0u;
            if (idx == a.N - 1) {
                a.rp[a.n] = a.N;
                if (a.rp_raw) a.rp_raw[a.n] = a.N;
                a.mark[a.n] = 1;
            }
        }
    }
    if (a.dups) {
        uint32_t x = ndup;
        for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
        if (lane == 0) s_dups[tid >> 6] = x;
        __syncthreads();
        if (tid == 0) {
            uint32_t t = 0;
            for (int i = 0; i < kPlainThreads / 64; ++i) t += s_dups[i];
            if (t) atomicAdd((unsigned long long *)a.dups, (unsigned long long)t);
        }
    }
}

// The kept entries of all earlier tiles, by a decoupled look-back in which one
// wavefront reads 64 predecessors per round trip: the nearest one with an
// inclusive prefix ends the walk, the counts of the ones before it are added.
// `tot` are the tile's own, published by one lane as early as they are known.
// (All 64 lanes call tile_prefix and get the prefix.)
__device__ __forceinline__ void tile_publish(const FinArgs &a, uint64_t tile, uint32_t tot) {
    store_agent(a.status + tile, status_word(1, tile == 0 ? kFlagIncl : kFlagAgg, tot));
}
__device__ __forceinline__ uint64_t tile_prefix(const FinArgs &a, uint64_t tile, uint32_t tot, uint32_t lane) {
    uint64_t *st = a.status + tile;
    uint64_t prefix = 0;
    if (tile > 0) {
        uint64_t j = tile;  // this step reads tiles j-1 .. j-64
        for (;;) {
            const bool real = j > lane;
            const uint64_t *pj = a.status + (real ? j - 1 - lane : 0);
            uint64_t v = real ? load_agent(pj) : status_word(1, kFlagIncl, 0);
            uint32_t spins = 0;
            while (status_tag(v) != 1u) {
                if (++spins > kSpinLimit || ((spins & 1023) == 0 && load_agent(a.err) != 0)) {
                    raise_device_error(a.err, DEVERR_LOOKBACK);
                    v = status_word(1, kFlagIncl, 0);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
                v = load_agent(pj);
            }
            const uint64_t incl = __ballot(status_flag(v) == kFlagIncl);
            const uint32_t first = incl ? (uint32_t)__builtin_ctzll(incl) : 64u;
            uint64_t c = lane <= first ? status_count(v) : 0;
            for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
            prefix += c;
            if (incl) break;
            j -= 64;  // j > 64 here: a lane past tile 0 reads an inclusive zero
        }
        if (lane == 0) store_agent(st, status_word(1, kFlagIncl, prefix + tot));
    }
    return prefix;
}

// One DPP instruction: the value of the lane below, lane 0 that of `first`.
__device__ __forceinline__ uint32_t lane_below(uint32_t v, uint32_t first) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)first, (int)v, 0x138 /*wave_shr:1*/, 0xF, 0xF, false);
}
__device__ __forceinline__ uint64_t lane_below(uint64_t v, uint64_t first) {
    return make_u64(lane_below((uint32_t)v, (uint32_t)first), lane_below((uint32_t)(v >> 32), (uint32_t)(first >> 32)));
}
__device__ __forceinline__ uint32_t last_lane(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, 63); }
__device__ __forceinline__ uint64_t last_lane(uint64_t v) {
    return make_u64(last_lane((uint32_t)v), last_lane((uint32_t)(v >> 32)));
}

// SIMPLE finish: keep the first of every run of equal entries unless it is a
// self-loop.  Output positions come from a look-back scan of the kept counts.
// A wave's keys are consecutive and stay in registers, item i of lane l being
// key 64 i + l: the entry before a key is the lane below's, kept entries are
// ranked by ballots, and the columns of an item leave as one run.  With the
// keys and then the kept columns staged through LDS, a thread's keys consecutive,
// 4.8e7 8-byte entries took 269 us (333 in tiles of 3,072), now 200: 0.82 GB, 4.1 TB/s.
template <typename IdT, typename KeyT>
__global__ __launch_bounds__(kFinThreads, 4) void csr_finish(FinArgs a) {
    constexpr int kWaves = kFinThreads / 64;
    __shared__ uint32_t s_counts[kWaves];  // kept entries of a wave | repeats << 16
    __shared__ uint64_t s_base;
    static_assert(kFinTile < (1 << 16), "a tile's counts fit 16 bits");
    const uint32_t lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint64_t tile = blockIdx.x;  // dispatch order (see radix_pass)
    const uint64_t base = tile * kFinTile + (uint64_t)w * 64 * kFinItems;  // of the wave
    const KeyT *K = static_cast<const KeyT *>(a.keys);
    const KeyT mask = ((KeyT)1 << a.wb) - 1;
    KeyT k[kFinItems];
    const uint32_t left = base < a.N ? (uint32_t)min(a.N - base, (uint64_t)(64 * kFinItems)) : 0u;  // of the wave's
    const KeyT *Kw = K + min(base, a.N - 1);
#pragma unroll
    for (int i = 0; i < kFinItems; ++i) k[i] = Kw[64 * i + lane < left ? 64 * i + lane : 0];
    KeyT before = base > 0 ? K[min(base, a.N) - 1] : ~Kw[0];  // (nothing is equal to, or in the row of, the one before the first)
    uint32_t keeps = 0, starts = 0, counts = 0;  // bit i: of item i
#pragma unroll
    for (int i = 0; i < kFinItems; ++i) {
        const KeyT key = k[i], prev = lane_below(key, before), row = key >> a.wb;
        before = last_lane(key);
        const bool in = 64 * i + lane < left, dup = key == prev;
        const bool keep = in & !dup & (row != (key & mask));
        counts += (uint32_t)__popcll(__ballot(keep)) | (uint32_t)__popcll(__ballot(in & dup)) << 16;
        keeps |= (uint32_t)keep << i;
        starts |= (uint32_t)(in & (row != (prev >> a.wb)) & ((uint64_t)row < a.n)) << i;
        // (decided here, and the row shifted out again below: of an item only the
        // key and two bits are held meanwhile)
        asm volatile("" : "+v"(keeps), "+v"(starts));
    }
    if (lane == 0) s_counts[w] = counts;
    __syncthreads();
    uint32_t all = 0, below = 0;
#pragma unroll
    for (int x = 0; x < kWaves; ++x) {
        below += x < w ? s_counts[x] : 0u;
        all += s_counts[x];
    }
    const uint32_t tot = all & 0xFFFFu;
    if (w == 0) {
        if (lane == 0) tile_publish(a, tile, tot);
        const uint64_t prefix = tile_prefix(a, tile, tot, lane);
        if (lane == 0) s_base = prefix;
    }
    __syncthreads();
    uint64_t c = s_base + (below & 0xFFFFu);
    IdT *col = static_cast<IdT *>(a.col);
#pragma unroll
    for (int i = 0; i < kFinItems; ++i) {
        const bool keep = (keeps >> i) & 1u;
        const uint64_t lanes = __ballot(keep);
        asm volatile("" : "+v"(k[i]));
        const uint64_t at = c + count_below(lanes);
        if ((starts >> i) & 1u) {
            const uint64_t row = (uint64_t)(k[i] >> a.wb);
            a.rp[row] = at;
            if (a.rp_raw) a.rp_raw[row] = base + 64 * i + lane;
            a.mark[row] = 1;
        }
        if (keep) __builtin_nontemporal_store((IdT)(k[i] & mask), &col[at]);
        c += (uint32_t)__popcll(lanes);
    }
    if (threadIdx.x == 0) {
        if (a.dups && (all >> 16)) atomicAdd((unsigned long long *)a.dups, (unsigned long long)(all >> 16));
        // The last tile closes row n.
        if ((tile + 1) * kFinTile >= a.N) {
            a.rp[a.n] = s_base + tot;
            if (a.rp_raw) a.rp_raw[a.n] = a.N;
            a.mark[a.n] = 1;
        }
    }
}

// The merged position of sorted random pair j: a power entry precedes the
// random pairs equal to it.
template <typename KeyT>
__device__ __forceinline__ uint64_t merged_position(const Power &p, const CountTables &t, const KeyT *R, uint64_t j, int wb) {
    const uint64_t key = R[j];
    bool member;
    return j + power_count(p.c, t, (uint32_t)(key >> wb), (uint32_t)(key & ((1ull << wb) - 1)), &member);
}

// split[t] for every tile boundary t = 0 .. tiles, by binary search.
template <typename KeyT>
__global__ __launch_bounds__(256) void xor_split(Power p, const KeyT *R, uint64_t random, uint64_t N, uint64_t tiles, int tile,
                                                 int wb, uint64_t *split) {
    __shared__ CountTables s_t;
    power_load(p, &s_t);
    __syncthreads();
    const uint64_t t = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (t > tiles) return;
    const uint64_t d = min(t * tile, N);
    uint64_t lo = d > p.entries ? d - p.entries : 0, hi = min(d, random);
    while (lo < hi) {
        const uint64_t mid = lo + (hi - lo) / 2;
        if (merged_position(p, s_t, R, mid, wb) < d)
            lo = mid + 1;
        else
            hi = mid;
    }
    split[t] = lo;
}

// XOR finish.  The sequence is the merge of a Kronecker power, whose entries are
// computed where they are needed (power.hpp), with the sorted pairs of a random
// graph, which may repeat; an origin bit below the entry (0 = power) puts the
// power's copy of a pair first; one copy of a pair present in exactly one of the
// two graphs is kept.
// Only the random pairs are sorted and read.  With the power's entries
// written as keys, sorted and read back as well, a graph of 2.1e8 + 1e8 entries
// took 13.5 ms, 10.4 of it in preparing, sorting and finishing 3.1e8 keys;
// merged, this kernel takes 2.3 ms and the sort 2.3.  It moves 1.7 GB (0.35 ms at
// the rate of a copy) and is bound by the walk's arithmetic and the latency of
// its table loads.  Counting what it keeps only after the walk made every tile
// wait for the slowest one in flight (3.0 ms; 2.4 with the counts published
// before it), and a walk that waited for each middle column itself 2.4.
template <typename IdT, typename RawT, int ITEMS>
__global__ __launch_bounds__(kXorThreads, 4) void csr_finish_xor(FinArgs a, Power pw) {
    constexpr int kThreads = kXorThreads, kItems = ITEMS, kTile = kThreads * kItems;
    using KeyT = uint64_t;
    // The walk writes kItems consecutive entries per thread, which would hit few
    // LDS banks across the wave; one pad slot per 16 entries spreads them.  Slot
    // 0 holds the entry before the tile, the last slot the one after it.
    __shared__ KeyT s_keys[kTile + kTile / 16 + 2];
    __shared__ int32_t s_change[kThreads / 64];
    __shared__ uint32_t s_tmp[kThreads / 64];
    __shared__ uint64_t s_base;
    const int tid = threadIdx.x;
    const uint64_t tile = blockIdx.x;  // dispatch order (see radix_pass)
    const uint64_t t0 = tile * kTile;
    __shared__ CountTables s_ct;
    __shared__ uint32_t s_taken[(kTile + 31) / 32 + 1];  // positions that hold a random pair
    const RawT *R = static_cast<const RawT *>(a.keys);
    power_load(pw, &s_ct);
    for (int i = tid; i < (kTile + 31) / 32 + 1; i += kThreads) s_taken[i] = 0;
    const uint64_t j0 = a.split[tile], j1 = a.split[tile + 1];
    __syncthreads();
    const uint64_t idmask = (1ull << a.wb) - 1;
    auto count_of = [&](uint64_t key, bool *member) {
        return power_count(pw.c, s_ct, (uint32_t)(key >> a.wb), (uint32_t)(key & idmask), member);
    };
    // The tile keeps its power entries, less those that a random pair takes out
    // (it follows them), plus the first copies of the other random pairs: known
    // from the random pairs alone, and published before the walk.
    int32_t change = 0;
    bool member;
    auto pack_at = [&](const PowerWalk &w) { return (((uint64_t)w.u << a.wb) | (w.rest + *w.mid * pw.w.midplace + *w.low)) << 1; };
    for (uint64_t jb = j0; jb < j1; jb += 4 * kThreads) {  // (the loads of a round go out together)
        uint64_t key[4], prev[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint64_t j = min(jb + i * kThreads + tid, j1 - 1);
            key[i] = R[j];
            prev[i] = R[j > 0 ? j - 1 : 0];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint64_t j = jb + i * kThreads + tid;
            if (j >= j1) break;
            const uint32_t x = (uint32_t)(j + count_of(key[i], &member) - t0);
            if (j == 0 || prev[i] != key[i]) change += member ? (x > 0 ? -1 : 0) : 1;
            s_keys[fin_slot(x + 1)] = (key[i] << 1) | 1u;
            atomicOr(&s_taken[x / 32], 1u << (x % 32));
        }
    }
    // The neighbours of the tile: either the random pair or the power
    // entry next to it.
    if (tid == 0) {
        uint64_t v = 0;
        if (t0 > 0) {
            const uint64_t g0 = t0 - j0;  // power entries before the tile
            const uint64_t key = j0 > 0 ? (uint64_t)R[j0 - 1] : 0;
            if (j0 > 0 && j0 - 1 + count_of(key, &member) == t0 - 1) {
                v = (key << 1) | 1u;
            } else {
                PowerWalk w;
                w.seek(pw.w, *pw.tables, g0 - 1);
                v = pack_at(w);
            }
        }
        s_keys[0] = v;
    }
    if (tid == 64) {
        uint64_t v = 0;
        const uint64_t t1 = t0 + kTile;
        if (t1 < a.N) {
            const uint64_t key = j1 < a.random ? (uint64_t)R[j1] : 0;
            if (j1 < a.random && j1 + count_of(key, &member) == t1) {
                v = (key << 1) | 1u;
                if (member && (j1 == 0 || (uint64_t)R[j1 - 1] != key)) --change;  // (its copy ends this tile)
            } else {
                PowerWalk w;
                w.seek(pw.w, *pw.tables, t1 - j1);
                v = pack_at(w);
            }
        }
        s_keys[fin_slot(kTile + 1)] = v;
    }
    for (int off = 32; off > 0; off >>= 1) change += __shfl_xor(change, off, 64);
    if ((tid & 63) == 0) s_change[tid >> 6] = change;
    __syncthreads();
    uint32_t all_kept = (uint32_t)(min(a.N - t0, (uint64_t)kTile) - (j1 - j0));
#pragma unroll
    for (int x = 0; x < kThreads / 64; ++x) all_kept += (uint32_t)s_change[x];
    if (tid == 0) tile_publish(a, tile, all_kept);
    // The power's entries take the other positions in order.
    {
        const int p0 = tid * kItems;
        const uint64_t two = (uint64_t)s_taken[p0 / 32] | ((uint64_t)s_taken[p0 / 32 + 1] << 32);
        const uint32_t taken = (uint32_t)(two >> (p0 % 32)) & ((1u << kItems) - 1);
        uint32_t all;
        const uint32_t before = block_exclusive_scan<kThreads>((uint32_t)__popc(taken), s_tmp, &all);
        // (the first wavefront looks back here, so that no tile waits for a
        // slower one's walk)
        if (tid < 64) {
            const uint64_t prefix = tile_prefix(a, tile, all_kept, tid);
            if (tid == 0) s_base = prefix;
        }
        uint64_t g = t0 - j0 + p0 - before;
        PowerWalk w;
        bool at = false;
        uint32_t row[kItems], rest[kItems], mid[kItems], low[kItems];  // (the loads of all items go out together)
#pragma unroll
        for (int j = 0; j < kItems; ++j) {
            row[j] = rest[j] = mid[j] = low[j] = 0;
            if (((taken >> j) & 1u) || t0 + p0 + j >= a.N) continue;
            if (at)
                w.next(pw.w, *pw.tables, g);
            else
                w.seek(pw.w, *pw.tables, g);
            at = true;
            ++g;
            row[j] = w.u;
            rest[j] = w.rest;
            mid[j] = *w.mid;
            low[j] = *w.low;
        }
#pragma unroll
        for (int j = 0; j < kItems; ++j)
            if (!((taken >> j) & 1u))
                s_keys[fin_slot(p0 + j + 1)] = (((uint64_t)row[j] << a.wb) | (rest[j] + mid[j] * pw.w.midplace + low[j])) << 1;
    }
    __syncthreads();
    // From here on a wave's entries are consecutive, item i of lane l being
    // entry 64 i + l (as in csr_finish).  eq: lanes whose pair equals the one
    // before it; an entry is kept if it is the first of its pair and either a
    // random pair or not followed by the same one.
    const uint32_t lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t p1 = (uint32_t)w * 64 * kItems;  // the wave's first entry in the tile
    const uint32_t left = (uint32_t)(t0 + p1 < a.N ? min(a.N - t0 - p1, (uint64_t)(64 * kItems)) : 0);
    const uint64_t mask = (1ull << a.wb) - 1;
    KeyT k[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) k[i] = s_keys[fin_slot(p1 + 64 * i + lane + 1)];
    KeyT before = t0 + p1 > 0 ? s_keys[fin_slot(p1)] : ~0ull;  // (no pair is as large)
    const KeyT after = s_keys[fin_slot(p1 + 64 * kItems + 1)];
    uint32_t keeps = 0, starts = 0, kept = 0;
    uint64_t eq = 0, first = 0;  // of the item before, whose keeping the next item's eq settles
    bool random = false;
#pragma unroll
    for (int i = 0; i <= kItems; ++i) {
        uint64_t eq_i = 0, first_i = 0;
        bool random_i = false;
        if (i < kItems) {
            const KeyT key = k[i], prev = lane_below(key, before);
            before = last_lane(key);
            const bool in = 64 * i + lane < left;
            eq_i = __ballot(in & ((key ^ prev) <= 1u));
            first_i = __ballot(in) & ~eq_i;
            random_i = key & 1u;
            const uint64_t row = key >> (a.wb + 1);
            starts |= (uint32_t)(in & (row != prev >> (a.wb + 1)) & (row < a.n)) << i;
        } else {
            eq_i = 64 * kItems <= left && t0 + p1 + 64 * kItems < a.N && (after ^ before) <= 1u;
        }
        if (i > 0) {
            const uint64_t lanes = first & (__ballot(random) | ~(eq >> 1 | eq_i << 63));
            kept += (uint32_t)__popcll(lanes);
            keeps |= (uint32_t)(lanes >> lane & 1u) << (i - 1);
        }
        eq = eq_i;
        first = first_i;
        random = random_i;
        asm volatile("" : "+v"(keeps), "+v"(starts));
    }
    if (lane == 0) s_tmp[w] = kept;
    __syncthreads();
    uint32_t below = 0;
#pragma unroll
    for (int x = 0; x < kThreads / 64; ++x) below += x < w ? s_tmp[x] : 0u;
    uint64_t c = s_base + below;
    IdT *col = static_cast<IdT *>(a.col);
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const bool keep = (keeps >> i) & 1u;
        const uint64_t lanes = __ballot(keep);
        asm volatile("" : "+v"(k[i]));
        const uint64_t at = c + count_below(lanes);
        if ((starts >> i) & 1u) {
            const uint64_t row = k[i] >> (a.wb + 1);
            a.rp[row] = at;
            a.mark[row] = 1;
        }
        if (keep) __builtin_nontemporal_store((IdT)(k[i] >> 1 & mask), &col[at]);
        c += (uint32_t)__popcll(lanes);
    }
    // The last tile closes row n.
    if (tid == 0 && t0 + kTile >= a.N) {
        a.rp[a.n] = s_base + all_kept;
        a.mark[a.n] = 1;
    }
}

// --------------------------------------------------------------------------- row fill
// mark[v] = 1 where rp[v] was written (a row with an entry; rp[n] always is).
// Afterwards every rp[v] holds the value of the first marked row at or after
// v.  Values at marked rows rise with the row, so that is a reverse running
// minimum, taken per chunk of kScanChunk rows: the first marked value of every
// chunk, an exclusive reverse scan over the chunks, then the chunk itself.
// Unmarked rows are written without being read, and only the marks are
// read for them.

// Marks of rows v0 .. v0+15 (v0 a multiple of 16) as a 16-bit mask.
__device__ __forceinline__ uint32_t load_marks16(const uint8_t *mark, uint64_t v0, uint64_t n1) {
    if (v0 + 16 <= n1) {
        const uint4 m = *reinterpret_cast<const uint4 *>(mark + v0);
        const uint32_t w[4] = {m.x, m.y, m.z, m.w};
        uint32_t bits = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int b = 0; b < 4; ++b) bits |= ((w[q] >> (8 * b)) & 1u) << (4 * q + b);
        return bits;
    }
    uint32_t bits = 0;
    for (uint64_t v = v0; v < n1; ++v) bits |= (uint32_t)(mark[v] & 1u) << (uint32_t)(v - v0);
    return bits;
}

// Degree bin: 0 for degree 0, b for 2^(b-1) <= d < 2^b, 31 above.
__device__ __forceinline__ int log2_bin(uint64_t d) {
    if (d == 0) return 0;
    const int b = 64 - __clzll(d);  // floor(log2 d) + 1
    return b > 31 ? 31 : b;
}

// The arrays of a row fill: row starts, then (with a histogram) the sorted
// positions' row starts and the column starts where the CSR has them.
struct FillArrays {
    struct One {
        uint64_t *A;
        const uint8_t *mark;
        uint64_t *cmin;  // [chunks]
        bool degree;     // A[v + 1] - A[v] counts towards the degree of v
    } a[3];
    int count, fills;    // arrays; the first `fills` of them are to be filled, the others only counted
    uint64_t n1, chunks;
    uint64_t *hist;
};

__global__ __launch_bounds__(256) void rowfill_first(FillArrays f) {
    __shared__ uint32_t s_first;
    if (threadIdx.x == 0) s_first = ~0u;
    __syncthreads();
    const FillArrays::One &a = f.a[blockIdx.y];
    constexpr int per = kScanChunk / 256;
    const uint64_t c0 = (uint64_t)blockIdx.x * kScanChunk;
    const uint64_t v0 = c0 + (uint64_t)threadIdx.x * per;
    const uint32_t bits = v0 < f.n1 ? load_marks16(a.mark, v0, f.n1) : 0u;
    if (bits) atomicMin(&s_first, (uint32_t)threadIdx.x * per + (uint32_t)__builtin_ctz(bits));
    __syncthreads();
    if (threadIdx.x == 0) a.cmin[blockIdx.x] = s_first == ~0u ? kNoRow : a.A[c0 + s_first];
}

// Exclusive reverse min-scan of the chunk minima (one block per array).  Thread t
// takes a contiguous range of whole kChunkBatch batches (128-byte aligned),
// moved by 16-byte vector loads and stores, so that the range is not walked
// one memory latency per chunk.
constexpr int kChunkBatch = 16;

__device__ __forceinline__ void load_batch(const uint64_t *p, uint64_t b, uint64_t hi, uint64_t (&x)[kChunkBatch]) {
    if (b + kChunkBatch <= hi) {
#pragma unroll
        for (int i = 0; i < kChunkBatch; i += 2) {
            const ulonglong2 v = *reinterpret_cast<const ulonglong2 *>(p + b + i);
            x[i] = v.x;
            x[i + 1] = v.y;
        }
    } else {
        for (int i = 0; i < kChunkBatch; ++i) x[i] = b + i < hi ? p[b + i] : kNoRow;
    }
}

__global__ __launch_bounds__(1024) void rowfill_chunks(FillArrays f) {
    __shared__ uint64_t s[1024];
    uint64_t *cmin = f.a[blockIdx.x].cmin;
    const uint64_t nchunks = f.chunks;
    const uint64_t per = ((nchunks + 1023) / 1024 + kChunkBatch - 1) / kChunkBatch * kChunkBatch;
    const uint64_t lo = min((uint64_t)threadIdx.x * per, nchunks), hi = min(lo + per, nchunks);
    const uint64_t nb = (hi - lo + kChunkBatch - 1) / kChunkBatch;
    uint64_t m = kNoRow;
    for (uint64_t k = 0; k < nb; ++k) {
        uint64_t x[kChunkBatch];
        load_batch(cmin, lo + k * kChunkBatch, hi, x);
#pragma unroll
        for (int i = 0; i < kChunkBatch; ++i) m = min(m, x[i]);
    }
    s[threadIdx.x] = m;
    __syncthreads();
    // inclusive suffix min over threads
    for (int off = 1; off < 1024; off <<= 1) {
        uint64_t other = threadIdx.x + off < 1024 ? s[threadIdx.x + off] : kNoRow;
        __syncthreads();
        s[threadIdx.x] = min(s[threadIdx.x], other);
        __syncthreads();
    }
    uint64_t run = threadIdx.x + 1 < 1024 ? s[threadIdx.x + 1] : kNoRow;
    // Backwards over the range: cmin[c] becomes the minimum over the chunks
    // after c.
    for (uint64_t k = nb; k-- > 0;) {
        const uint64_t b = lo + k * kChunkBatch;
        uint64_t x[kChunkBatch], y[kChunkBatch];
        load_batch(cmin, b, hi, x);
#pragma unroll
        for (int i = kChunkBatch - 1; i >= 0; --i) {
            y[i] = run;
            if (b + i < hi) run = min(run, x[i]);
        }
        if (b + kChunkBatch <= hi) {
#pragma unroll
            for (int i = 0; i < kChunkBatch; i += 2) {
                ulonglong2 v;
                v.x = y[i];
                v.y = y[i + 1];
                *reinterpret_cast<ulonglong2 *>(cmin + b + i) = v;
            }
        } else {
            for (int i = 0; i < kChunkBatch; ++i)
                if (b + i < hi) cmin[b + i] = y[i];
        }
    }
}

// The marks of rows v0 .. v0+3 (v0 a multiple of 4).
__device__ __forceinline__ uint32_t load_marks4(const uint8_t *mark, uint64_t v0, uint64_t n1) {
    uint32_t bits = 0;
    if (v0 + 4 <= n1) {
        const uint32_t m = *reinterpret_cast<const uint32_t *>(mark + v0);
#pragma unroll
        for (int b = 0; b < 4; ++b) bits |= ((m >> (8 * b)) & 1u) << b;
    } else {
        for (uint64_t v = v0; v < n1; ++v) bits |= (uint32_t)(mark[v] & 1u) << (uint32_t)(v - v0);
    }
    return bits;
}

// The first marked value at or after row v (a multiple of 16); kNoRow if there
// is none.  Whole workgroup of 256, 16,384 rows per step; marked rows only ever
// hold their final value.
__device__ __forceinline__ uint64_t marked_from(const FillArrays::One &a, uint64_t v, uint64_t n1, uint32_t *s_first) {
    constexpr int kAhead = 4;
    for (; v < n1; v += 256 * 16 * kAhead) {
        uint32_t bits[kAhead];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const uint64_t v0 = v + (uint64_t)(q * 256 + (int)threadIdx.x) * 16;
            bits[q] = v0 < n1 ? load_marks16(a.mark, v0, n1) : 0u;
        }
        uint32_t mine = ~0u;
#pragma unroll
        for (int q = kAhead - 1; q >= 0; --q)
            if (bits[q]) mine = (uint32_t)(q * 256 + (int)threadIdx.x) * 16 + (uint32_t)__builtin_ctz(bits[q]);
        if (threadIdx.x == 0) *s_first = ~0u;
        __syncthreads();
        if (mine != ~0u) atomicMin(s_first, mine);
        __syncthreads();
        const uint32_t first = *s_first;
        __syncthreads();
        if (first != ~0u) return a.A[v + first];
    }
    return kNoRow;
}

// One chunk of every array.  HIST: the degree histogram (the degrees of the
// paper's Results section) over rows v < n1 - 1 is counted from the filled
// values, the degree of v being the sum of A[v+1] - A[v] over the arrays that
// count towards it.  SELF: the value after the chunk is looked for in the
// marks here, not taken from the chunk scan, and the chunks are shorter: such a
// fill has few of them, and each takes as long as its serial steps.  REST: the
// arrays from f.fills on have been filled before and are read for the degrees (as a
// flag of the array it cost every fill with a histogram 9%).
constexpr int kSelfChunk = 1024;

template <bool HIST, bool SELF, bool REST = false> __global__ __launch_bounds__(256) void rowfill_apply(FillArrays f) {
    constexpr int kChunk = SELF ? kSelfChunk : kScanChunk, per = kChunk / 256;
    // Thread t owns rows t*per .. t*per+per-1 of the chunk; the results go
    // through LDS (one pad word per `per`) so the stores are coalesced.
    __shared__ uint64_t s_out[kChunk + kChunk / per];
    __shared__ uint64_t s_wave[4];
    __shared__ uint32_t s_h[32];
    __shared__ uint32_t s_first;
    const int tid = threadIdx.x;
    const uint32_t lane = tid & 63;
    const uint64_t n1 = f.n1, c0 = (uint64_t)blockIdx.x * kChunk;
    const uint64_t v0 = c0 + (uint64_t)tid * per;
    if (HIST && tid < 32) s_h[tid] = 0;
    uint64_t deg[HIST ? per : 1];  // of row c0 + 256 j + tid
    if (HIST)
#pragma unroll
        for (int j = 0; j < per; ++j) deg[j] = 0;
    if (HIST && REST)
        for (int q = f.fills; q < f.count; ++q) {
            const FillArrays::One &a = f.a[q];
            if (!a.degree) continue;
#pragma unroll
            for (int j = 0; j < per; ++j) {
                const uint64_t v = c0 + 256 * j + tid;
                if (v + 1 < n1) deg[j] += a.A[v + 1] - a.A[v];
            }
        }
    for (int q = 0; q < (REST ? f.fills : f.count); ++q) {
        const FillArrays::One &a = f.a[q];
        const uint32_t bits = v0 >= n1 ? 0u : SELF ? load_marks4(a.mark, v0, n1) : load_marks16(a.mark, v0, n1);
        uint64_t x[per];
        uint64_t m = kNoRow;
#pragma unroll
        for (int j = 0; j < per; ++j) {
            x[j] = ((bits >> j) & 1u) ? a.A[v0 + j] : kNoRow;  // marked rows only
            m = min(m, x[j]);
        }
        // the first marked value after the chunk
        const uint64_t next = SELF ? marked_from(a, c0 + kChunk, n1, &s_first) : a.cmin[blockIdx.x];
        // minimum over the rows of the threads after this one
        for (int off = 1; off < 64; off <<= 1) {
            const uint64_t o = __shfl_down(m, off, 64);
            if (lane + off < 64) m = min(m, o);
        }
        if (lane == 0) s_wave[tid >> 6] = m;
        __syncthreads();
        const uint64_t after = __shfl_down(m, 1, 64);
        uint64_t run = min(next, lane < 63 ? after : kNoRow);
        for (int w = (tid >> 6) + 1; w < 4; ++w) run = min(run, s_wave[w]);
#pragma unroll
        for (int j = per - 1; j >= 0; --j) {
            run = min(run, x[j]);
            s_out[tid * (per + 1) + j] = run;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < per; ++j) {
            const int i = 256 * j + tid;
            const uint64_t v = c0 + i;
            const uint64_t a0 = s_out[(i / per) * (per + 1) + i % per];
            if (v < n1) a.A[v] = a0;
            if (HIST && a.degree && v + 1 < n1)  // the row after the chunk's last holds `next` once filled
                deg[j] += (i + 1 < kChunk ? s_out[((i + 1) / per) * (per + 1) + (i + 1) % per] : next) - a0;
        }
        __syncthreads();  // s_wave and s_out are rewritten for the next array
    }
    if (HIST) {
#pragma unroll
        for (int j = 0; j < per; ++j) {
            const bool row = c0 + 256 * j + tid + 1 < n1;
            const int b = row ? log2_bin(deg[j]) : 0;
            // Most vertices of a scale-free graph have small degree: bin 0
            // is counted by ballot, the rest by LDS atomics.
            const uint64_t zero = __ballot(row && b == 0);
            if (lane == 0 && zero) atomicAdd(&s_h[0], (uint32_t)__popcll(zero));
            if (row && b != 0) atomicAdd(&s_h[b], 1u);
        }
        __syncthreads();
        if (tid < 32 && s_h[tid]) atomicAdd((unsigned long long *)&f.hist[tid], (unsigned long long)s_h[tid]);
    }
}

// --------------------------------------------------------------------------- host
int bits_for(uint64_t n) {  // bits to hold ids in [0, n)
    int b = 1;
    while (b < 64 && (n - 1) >> b) ++b;
    return b;
}

constexpr uint64_t tiles_of(uint64_t entries, int items) {
    return (entries + kPassThreads * items - 1) / (kPassThreads * items);
}
constexpr int pass_items(uint64_t entries) {
    return entries <= kShortTiles * kPassThreads * kShortItems ? kShortItems : entries <= kShortList ? kMidItems : kPassItems;
}
// Bytes of the passes' look-back words that a list uses, and that its plan has.
constexpr uint64_t words_used(uint64_t entries) {
    const int items = pass_items(entries);
    return tiles_of(entries, items) * kRadix * (items < kPassItems ? sizeof(uint32_t) : sizeof(uint64_t));
}
constexpr uint64_t words_reserved(uint64_t entries) {
    return ((entries ? tiles_of(entries, kPassItems) : 1) + kSpareTiles) * kRadix * sizeof(uint64_t);
}
constexpr bool words_fit() {
    for (uint64_t n = 0; n <= kShortList + 1; n += kPassThreads)
        for (uint64_t e : {n, n + 1})
            if (words_used(e) > words_reserved(e)) return false;
    return true;
}
static_assert(words_fit(), "no list uses more look-back words than its plan has (checked around every tile's edge)");

struct Plan {
    uint64_t n, E, N;
    int wb, db, kb, passes, key_bytes, dpasses;
    bool sym, simple, hist, directed_hist, xor_mode;
    bool fused_finish;  // the last pass writes the CSR (FINAL) instead of keys
    uint64_t power;  // (XOR) entries of the Kronecker power, beside the N sorted ones
    int items;  // keys per thread of the digit passes' tiles
    int xor_items;  // entries per thread of the XOR finish's tiles
    uint64_t pass_tiles, fin_tiles, chunks;
    // workspace carving
    size_t off_keysA, off_keysB, off_status, off_ghist, off_gbase, off_indeg, off_rpraw, off_mark,  // in this order
        off_cmark, off_cmin, off_fstatus, off_split, off_tables, total;
};

Plan make_plan(uint64_t n, uint64_t E, int id_bytes, uint32_t flags, bool want_hist, bool xor_mode = false,
               uint64_t power = 0) {
    Plan p;
    memset(&p, 0, sizeof(p));
    p.n = n;
    p.E = E;
    p.sym = flags & SFG_CSR_SYMMETRIZE;
    p.simple = (flags & SFG_CSR_SIMPLE) || xor_mode;
    p.xor_mode = xor_mode;
    p.power = power;
    p.N = p.sym ? 2 * E : E;
    p.wb = bits_for(n);
    p.hist = want_hist;
    p.directed_hist = want_hist && !p.sym;
    // With in-degrees wanted, the destination field fills whole digits so
    // that some pass boundary leaves the keys ordered by destination.
    p.db = p.directed_hist ? 8 * ((p.wb + 7) / 8) : p.wb;
    // Symmetrized: a whole-byte destination field lets the histogram pass
    // count bytes of the two endpoints instead of every digit of both keys;
    // taken when it costs no pass and no key width.
    if (p.sym) {
        const int db8 = 8 * ((p.wb + 7) / 8);
        if ((p.wb + db8 + 7) / 8 == (2 * p.wb + 7) / 8 && (p.wb + db8 <= 32) == (2 * p.wb <= 32)) p.db = db8;
    }
    p.dpasses = p.db / 8;
    p.kb = p.wb + p.db;
    p.passes = (p.kb + 7) / 8;
    p.key_bytes = p.kb <= 32 ? 4 : 8;
    p.items = pass_items(p.N);
    p.pass_tiles = tiles_of(p.N, p.items);
    p.xor_items = xor_items(p.N + power);
    p.fin_tiles = xor_mode ? xor_tiles(p.N + power, p.xor_items) : (p.N + kFinTile - 1) / kFinTile;
    // Without SIMPLE no entry is dropped, so sorted positions are output
    // positions and the last pass can write the columns itself -- unless it
    // is also the first pass or the pass that marks column starts.
    p.fused_finish = !p.simple && p.passes >= 2 && !(p.directed_hist && p.passes - 1 == p.dpasses);
    p.chunks = (n + 1 + kScanChunk - 1) / kScanChunk;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        size_t r = o;
        o += align256(bytes);
        return r;
    };
    // keysA also holds the run records of a FINAL pass (first and last key
    // of every tile's run of every digit, and each tile's repeat count).
    const uint64_t records = p.fused_finish ? 2 * p.pass_tiles * kRadix * p.key_bytes + 4 * p.pass_tiles : 0;
    p.off_keysA = take(std::max<uint64_t>(p.N * p.key_bytes, records));
    p.off_keysB = take(p.N * p.key_bytes);
    p.off_status = take(words_reserved(p.N));
    p.off_ghist = take(8 * kRadix * 8);
    p.off_gbase = take(kRadix * 8);
    p.off_indeg = take(p.directed_hist ? (n + 1) * 8 : 0);
    p.off_rpraw = take(want_hist && p.simple ? (n + 1) * 8 : 0);
    p.off_mark = take(n + 1);
    p.off_cmark = take(p.directed_hist ? n + 1 : 0);
    p.off_cmin = take(std::max<uint64_t>(p.chunks, 1) * 8);
    // (XOR: room for as many tiles as any fewer entries have)
    uint64_t most = std::max<uint64_t>(p.fin_tiles, 1);
    if (xor_mode)
        most = std::max({most, xor_tiles(std::min(p.N + power, kXorShort), kXorShortItems),
                         xor_tiles(std::min(p.N + power, kXorMid), kXorMidItems)});
    p.off_fstatus = take(p.simple ? most * 8 : 0);
    p.off_split = take(xor_mode ? (most + 1) * 8 : 0);
    p.off_tables = take(xor_mode ? sizeof(PowerTables) : 0);
    p.total = o;
    (void)id_bytes;
    return p;
}

int fill_grid(uint64_t n) {
    const uint64_t want = (n + 255) / 256;
    return (int)std::max<uint64_t>(1, std::min<uint64_t>(want, (uint64_t)device_cu_count() * 8));
}

// Everything a build starts from, in one launch (a fill kernel, so the
// sequence stays valid under stream capture): the counters, histograms and
// look-back words zeroed, the marks zeroed except that of row n, and the
// values at row n.  A launch per region was half of a small graph's time.
struct ClearArgs {
    struct Region {
        uint4 *p;        // 16-byte aligned, its length rounded up to 16 bytes
        uint64_t words;  // 16-byte words
        uint64_t one;    // byte that is 1 instead of 0, or ~0
    } r[8];
    struct Value {
        uint64_t *p;
        uint64_t v;
    } v[4];
    int regions, values;
    uint64_t *hist;  // [32], the caller's (8-byte aligned), or null
    void region(void *p, uint64_t bytes, uint64_t one = ~0ull) { r[regions++] = {static_cast<uint4 *>(p), (bytes + 15) / 16, one}; }
    void value(uint64_t *p, uint64_t x) { v[values++] = {p, x}; }
};

__global__ __launch_bounds__(256) void csr_clear(ClearArgs a) {
    const uint64_t i0 = (uint64_t)blockIdx.x * 256 + threadIdx.x, stride = (uint64_t)gridDim.x * 256;
    for (int q = 0; q < a.regions; ++q) {
        const uint64_t at = a.r[q].one;  // (~0 / 16 is no word of any region)
        for (uint64_t i = i0; i < a.r[q].words; i += stride) {
            uint4 z = {0, 0, 0, 0};
            if (i == at / 16) {
                const uint32_t w = (uint32_t)(at / 4) % 4, x = 1u << (8 * (uint32_t)(at % 4));
                z = {w == 0 ? x : 0, w == 1 ? x : 0, w == 2 ? x : 0, w == 3 ? x : 0};
            }
            a.r[q].p[i] = z;
        }
    }
    if (i0 < (uint64_t)a.values) *a.v[i0].p = a.v[i0].v;
    if (a.hist && i0 < 32) a.hist[i0] = 0;
}

// The row fill of up to three arrays.  Up to kSelfChunks chunks the marks
// after a chunk are scanned by its own workgroup, one launch instead of three
// (eight steps in the worst case, against two launches of about 4 us).  The fill
// in us with rows all over / in the first five alone: 11.1 / 11.8 at 65,537
// vertices and 11.3 / 17.4 at 131,000, by three launches 20.8 / 19.4 and 20.3 / 18.9;
// at 16,384 vertices 10.2 in chunks of 1,024 rows, 14.2 in chunks of 4,096.
constexpr uint64_t kSelfChunks = 32;

void row_fill(const FillArrays &f, hipStream_t s) {
    ProfScope _ps("csr_rowfill", s);
    const unsigned g = (unsigned)f.chunks;
    if (f.chunks <= kSelfChunks) {
        const unsigned gs = (unsigned)((f.n1 + kSelfChunk - 1) / kSelfChunk);
        if (f.hist)
            rowfill_apply<true, true><<<gs, 256, 0, s>>>(f);
        else
            rowfill_apply<false, true><<<gs, 256, 0, s>>>(f);
        return;
    }
    rowfill_first<<<dim3(g, f.fills), 256, 0, s>>>(f);
    rowfill_chunks<<<f.fills, 1024, 0, s>>>(f);
    if (f.hist && f.fills < f.count)
        rowfill_apply<true, false, true><<<g, 256, 0, s>>>(f);
    else if (f.hist)
        rowfill_apply<true, false><<<g, 256, 0, s>>>(f);
    else
        rowfill_apply<false, false><<<g, 256, 0, s>>>(f);
}

// The key array the first pass reads when the keys are given (the passes
// ping-pong so that the last one writes keysA).
size_t first_input_offset(const Plan &P) { return (P.passes - 1) % 2 == 0 ? P.off_keysB : P.off_keysA; }

// counted: the workspace is cleared and the digit histograms are in it
// (counted by the producer of the edges), so the histogram pass is skipped.  keys_given: the
// producer also wrote every entry's key at first_input_offset, so the first
// pass reads keys like any other.
// Columns of a CSR over packed ids are unpacked by the last pass.
struct Unpack {
    const uint32_t *dec;
    int groups, bits;
};

// Clears what a build of this plan starts from (see ClearArgs).
void clear_csr(const Plan &P, uint64_t *row_ptr, uint64_t *hist, uint64_t *dups, char *ws, hipStream_t s) {
    ClearArgs c;
    memset(&c, 0, sizeof(c));
    uint64_t words = 0;
    auto region = [&](size_t off, uint64_t bytes, uint64_t one = ~0ull) {
        c.region(ws + off, bytes, one);
        words = std::max(words, c.r[c.regions - 1].words);
    };
    region(P.off_ghist, 8 * kRadix * 8);
    if (P.N) region(P.off_status, words_used(P.N));
    if (P.simple && P.fin_tiles) region(P.off_fstatus, P.fin_tiles * 8);
    // Row (and column) starts are written only where a row begins and
    // flagged in the mark bytes; the row fill completes the rest.
    region(P.off_mark, P.n + 1, P.n);
    if (P.directed_hist) {
        region(P.off_cmark, P.n + 1, P.n);
        c.value(reinterpret_cast<uint64_t *>(ws + P.off_indeg) + P.n, P.N);
    }
    c.hist = hist;
    if (dups) c.value(dups, 0);
    // (the last pass over the entries writes row n's value: the edge list, which
    // may share memory with row_ptr, has been read by then)
    if (P.N + P.power == 0) c.value(row_ptr + P.n, 0);
    if (P.hist && P.simple && P.N == 0) c.value(reinterpret_cast<uint64_t *>(ws + P.off_rpraw) + P.n, 0);
    ProfScope _ps("fill", s);
    csr_clear<<<fill_grid(words), 256, 0, s>>>(c);
}

template <typename IdT, typename KeyT, bool SYM, bool FIRST, bool BOUND, bool FINAL>
void launch_pass(const PassArgs &a, int grid, int items, hipStream_t s) {
    ProfScope _ps("radix_pass", s);
    if (items == kShortItems)
        radix_pass<IdT, KeyT, SYM, FIRST, BOUND, FINAL, kShortItems><<<grid, kPassThreads, 0, s>>>(a);
    else if (items == kMidItems)
        radix_pass<IdT, KeyT, SYM, FIRST, BOUND, FINAL, kMidItems><<<grid, kPassThreads, 0, s>>>(a);
    else
        radix_pass<IdT, KeyT, SYM, FIRST, BOUND, FINAL, kPassItems><<<grid, kPassThreads, 0, s>>>(a);
}

template <typename IdT, typename KeyT>
int run_csr(const Plan &P, const void *src, const void *dst, uint64_t *row_ptr, void *col, uint64_t *hist,
            uint64_t *dups, char *ws, hipStream_t s, bool counted = false, bool keys_given = false,
            const Unpack *up = nullptr, const Power *pw = nullptr) {
    uint32_t *err = device_error_word();
    KeyT *keysA = reinterpret_cast<KeyT *>(ws + P.off_keysA);
    KeyT *keysB = reinterpret_cast<KeyT *>(ws + P.off_keysB);
    uint64_t *status = reinterpret_cast<uint64_t *>(ws + P.off_status);
    uint64_t *ghist = reinterpret_cast<uint64_t *>(ws + P.off_ghist);
    uint64_t *gbase = reinterpret_cast<uint64_t *>(ws + P.off_gbase);
    uint64_t *csc = P.directed_hist ? reinterpret_cast<uint64_t *>(ws + P.off_indeg) : nullptr;
    uint64_t *rp_raw_ws = (P.hist && P.simple) ? reinterpret_cast<uint64_t *>(ws + P.off_rpraw) : nullptr;
    uint8_t *mark = reinterpret_cast<uint8_t *>(ws + P.off_mark);
    uint8_t *cmark = P.directed_hist ? reinterpret_cast<uint8_t *>(ws + P.off_cmark) : nullptr;
    uint64_t *fstatus = P.simple ? reinterpret_cast<uint64_t *>(ws + P.off_fstatus) : nullptr;
    if (!counted) clear_csr(P, row_ptr, hist, dups, ws, s);

    if (P.N > 0) {
        PrepArgs pa{P.E, P.N, src, dst, ghist, P.db, P.passes, (P.sym && P.db % 8 == 0) ? P.db / 8 : 0};
        // Every histogram workgroup stays resident (128 KB of LDS each); a small
        // list takes fewer, since each adds its counts to the global ones.
        const int pg = (int)std::max<uint64_t>(1, std::min<uint64_t>((P.E + kPrepMinEdges - 1) / kPrepMinEdges,
                                                                      (uint64_t)device_cu_count() * kPrepBlocksPerCu));
        if (!counted) {
            ProfScope _ps("csr_prepare", s);
            if (P.sym)
                csr_prepare<IdT, KeyT, true><<<pg, kPrepThreads, 0, s>>>(pa);
            else
                csr_prepare<IdT, KeyT, false><<<pg, kPrepThreads, 0, s>>>(pa);
        }
        // Ping-pong so that the last pass lands in keysA.
        for (int p = 0; p < P.passes; ++p) {
            const int remaining = P.passes - 1 - p;  // passes after this one
            KeyT *out = (remaining % 2 == 0) ? keysA : keysB;
            KeyT *in = (remaining % 2 == 0) ? keysB : keysA;
            PassArgs a{P.E, P.N, src, dst, in, out, status, gbase, ghist + p * kRadix, err,
                       csc, cmark, P.db, 8 * p, (uint32_t)(p + 1), P.n};
            const int g = (int)P.pass_tiles;
            if (P.fused_finish && p == P.passes - 1) {
                a.col = col;
                a.rp = row_ptr;
                a.mark = mark;
                a.run_first = out;
                a.run_last = out + P.pass_tiles * kRadix;
                a.tile_dups = reinterpret_cast<uint32_t *>(out + 2 * P.pass_tiles * kRadix);
                if (up) {
                    a.dec = up->dec;
                    a.dec_groups = up->groups;
                    a.dec_bits = up->bits;
                }
                launch_pass<IdT, KeyT, false, false, false, true>(a, g, P.items, s);
            } else if (csc && p == P.dpasses) {
                launch_pass<IdT, KeyT, false, false, true, false>(a, g, P.items, s);
            } else if (p == 0 && !keys_given) {
                if (P.sym)
                    launch_pass<IdT, KeyT, true, true, false, false>(a, g, P.items, s);
                else
                    launch_pass<IdT, KeyT, false, true, false, false>(a, g, P.items, s);
            } else {
                launch_pass<IdT, KeyT, false, false, false, false>(a, g, P.items, s);
            }
        }
    }
    const uint64_t entries = P.N + P.power;
    FinArgs fa{entries, P.n, keysA, col, row_ptr, P.simple ? rp_raw_ws : nullptr, mark, dups, fstatus, err, P.db,
               P.N, reinterpret_cast<const uint64_t *>(ws + P.off_split)};
    if (entries == 0) {
        // (the clearing kernel wrote the values at row n)
    } else if (P.fused_finish) {
        const int last = P.passes - 1;
        const int run_tiles = P.pass_tiles >= (uint64_t)kRunTiles * device_cu_count() ? kRunTiles : kRunBatch;
        RunArgs ra{P.pass_tiles, P.n, status, gbase, ghist + last * kRadix, keysA,
                   keysA + P.pass_tiles * kRadix, reinterpret_cast<const uint32_t *>(keysA + 2 * P.pass_tiles * kRadix),
                   row_ptr, P.N, mark, dups, err, P.db, (uint32_t)(last + 1), run_tiles};
        const int rg = (int)((P.pass_tiles + run_tiles - 1) / run_tiles);
        ProfScope _ps("csr_run_starts", s);
        if (P.items < kPassItems)
            csr_run_starts<KeyT, uint32_t><<<rg, kRadix, 0, s>>>(ra);
        else
            csr_run_starts<KeyT, uint64_t><<<rg, kRadix, 0, s>>>(ra);
    } else if (P.xor_mode) {
        ProfScope _ps("csr_finish", s);
        xor_split<KeyT><<<(int)((P.fin_tiles + 256) / 256), 256, 0, s>>>(
            *pw, keysA, P.N, entries, P.fin_tiles, kXorThreads * P.xor_items, P.db, reinterpret_cast<uint64_t *>(ws + P.off_split));
        if (P.xor_items == kXorItems)
            csr_finish_xor<IdT, KeyT, kXorItems><<<(int)P.fin_tiles, kXorThreads, 0, s>>>(fa, *pw);
        else if (P.xor_items == kXorMidItems)
            csr_finish_xor<IdT, KeyT, kXorMidItems><<<(int)P.fin_tiles, kXorThreads, 0, s>>>(fa, *pw);
        else
            csr_finish_xor<IdT, KeyT, kXorShortItems><<<(int)P.fin_tiles, kXorThreads, 0, s>>>(fa, *pw);
    } else if (P.simple) {
        ProfScope _ps("csr_finish", s);
        csr_finish<IdT, KeyT><<<(int)P.fin_tiles, kFinThreads, 0, s>>>(fa);
    } else {
        ProfScope _ps("csr_finish", s);
        csr_finish_plain<IdT, KeyT><<<fill_grid(P.N), kPlainThreads, 0, s>>>(fa);
    }
    // The degree histogram is counted by the fill: deg = out (from the
    // uncompacted row starts) + in (from the column starts, directed).
    FillArrays f;
    memset(&f, 0, sizeof(f));
    f.n1 = P.n + 1;
    f.chunks = P.chunks;
    f.hist = hist;
    auto add = [&](uint64_t *A, const uint8_t *m, bool degree) { f.a[f.count++] = {A, m, nullptr, degree}; };
    add(row_ptr, mark, hist && !rp_raw_ws);
    if (rp_raw_ws) add(rp_raw_ws, mark, true);
    if (csc) add(csc, cmark, true);
    // The chunk scans of a second and third array go where the keys and the
    // look-back words were (8 bytes per 4,096 rows): nothing reads those any more.
    f.a[0].cmin = reinterpret_cast<uint64_t *>(ws + P.off_cmin);
    const uint64_t cpad = (P.chunks + kChunkBatch - 1) / kChunkBatch * kChunkBatch;  // (vector loads)
    f.a[1].cmin = reinterpret_cast<uint64_t *>(ws + P.off_keysA);
    f.a[2].cmin = f.a[1].cmin + cpad;
    static_assert(kSelfChunks * 8 * 2 <= kSpareTiles * kRadix * 8, "a fill without a chunk scan needs no room");
    f.fills = f.count;
    if ((uint64_t)(f.count - 1) * cpad * 8 > P.off_indeg - P.off_keysA) {
        // (a few entries over 8 million rows or more: one array after the other, the last
        // one's launch reading the others' degrees)
        f.fills = 1;
        const int last = f.count - 1;
        for (int q = 0; q < last; ++q) {
            FillArrays one = f;
            one.a[0] = f.a[q];
            one.a[0].cmin = f.a[0].cmin;
            one.count = 1;
            one.hist = nullptr;
            row_fill(one, s);
        }
        uint64_t *cmin = f.a[0].cmin;
        std::swap(f.a[0], f.a[last]);
        f.a[0].cmin = cmin;
    }
    row_fill(f, s);
    return check_launch("edges_to_csr");
}

}  // namespace
}  // namespace sfg

using namespace sfg;

extern "C" size_t edges_to_csr_workspace_bytes(uint64_t n, uint64_t num_edges, int id_bytes, uint32_t flags) {
    return sfg::csr_workspace_bytes(n, num_edges, id_bytes, flags);
}

namespace sfg {

size_t csr_workspace_bytes(uint64_t n, uint64_t num_edges, int id_bytes, uint32_t flags) {
    if (n == 0) return 0;
    // With the histogram or without it: a small directed list takes more without,
    // since its shorter keys then let the last pass write the CSR, whose run records
    // are longer than a few keys.
    return std::max(make_plan(n, num_edges, id_bytes, flags, true).total, make_plan(n, num_edges, id_bytes, flags, false).total);
}

// The argument checks of edges_to_csr; on success P is its plan.
int csr_check(uint64_t n, uint64_t num_edges, const void *src, const void *dst, int id_bytes, uint32_t flags,
              const uint64_t *row_ptr, const void *col, const uint64_t *degree_hist32, const void *workspace,
              size_t workspace_bytes, Plan &P) {
    if (n == 0) return fail(SFG_EINVAL, "edges_to_csr: n must be >= 1");
    if (id_bytes != 4 && id_bytes != 8) return fail(SFG_EINVAL, "edges_to_csr: id_bytes must be 4 or 8");
    if (flags & ~(uint32_t)(SFG_CSR_SYMMETRIZE | SFG_CSR_SIMPLE)) return fail(SFG_EINVAL, "edges_to_csr: bad flags");
    if (!row_ptr) return fail(SFG_EINVAL, "edges_to_csr: row_ptr is NULL");
    if (num_edges > 0 && (!src || !dst || !col)) return fail(SFG_EINVAL, "edges_to_csr: NULL edge or col buffer");
    if (id_bytes == 4 && n - 1 > 0x7FFFFFFFull) return fail(SFG_ERANGE, "edges_to_csr: n does not fit int32 ids");
    if (n > (1ull << 32)) return fail(SFG_ERANGE, "edges_to_csr: n > 2^32 does not fit a 64-bit key");
    if (num_edges > (1ull << 54)) return fail(SFG_ERANGE, "edges_to_csr: too many edges");
    const bool sym = flags & SFG_CSR_SYMMETRIZE;
    const uint64_t N = sym ? 2 * num_edges : num_edges;
    // One workgroup per tile: a dispatch's work-item count must stay below 2^32
    // (2^34 entries are 2^21 digit-pass tiles of 1,024 threads, and 2^21 finish
    // tiles of 512).
    if (N > (1ull << 34)) return fail(SFG_ERANGE, "edges_to_csr: more than 2^34 entries");
    P = make_plan(n, num_edges, id_bytes, flags, degree_hist32 != nullptr);
    if (P.total > 0 && !workspace) return fail(SFG_EINVAL, "edges_to_csr: workspace is NULL");
    if (workspace_bytes < P.total)
        return fail(SFG_ENOSPACE, "edges_to_csr: workspace has %zu bytes, needs %zu", workspace_bytes, P.total);
    if (!device_error_word()) return fail(SFG_EDEVICE, "edges_to_csr: no device");
    return SFG_OK;
}

int csr_run(const Plan &P, const void *src, const void *dst, int id_bytes, uint64_t *row_ptr, void *col,
            uint64_t *degree_hist32, uint64_t *num_duplicates, char *ws, hipStream_t s, bool counted,
            bool keys_given = false, const Unpack *up = nullptr) {
    uint64_t *h = degree_hist32, *d = num_duplicates;
    if (P.key_bytes == 4) {
        // (4-byte keys are given only by a packing producer)
        if (id_bytes == 4) return run_csr<int32_t, uint32_t>(P, src, dst, row_ptr, col, h, d, ws, s, counted, up && keys_given, up);
        return run_csr<int64_t, uint32_t>(P, src, dst, row_ptr, col, h, d, ws, s, counted, up && keys_given, up);
    }
    if (id_bytes == 4) return run_csr<int32_t, uint64_t>(P, src, dst, row_ptr, col, h, d, ws, s, counted, keys_given, up);
    return run_csr<int64_t, uint64_t>(P, src, dst, row_ptr, col, h, d, ws, s, counted, keys_given, up);
}

int csr_build(uint64_t n, uint64_t num_edges, const void *src, const void *dst, int id_bytes, uint32_t flags,
              uint64_t *row_ptr, void *col, uint64_t *degree_hist32, uint64_t *num_duplicates, void *workspace,
              size_t workspace_bytes, hipStream_t s, const uint64_t **raw_rows) {
    Plan P;
    const int rc = csr_check(n, num_edges, src, dst, id_bytes, flags, row_ptr, col, degree_hist32, workspace,
                             workspace_bytes, P);
    if (rc != SFG_OK) return rc;
    char *ws = static_cast<char *>(workspace);
    if (raw_rows) *raw_rows = (P.hist && P.simple) ? reinterpret_cast<const uint64_t *>(ws + P.off_rpraw) : row_ptr;
    return csr_run(P, src, dst, id_bytes, row_ptr, col, degree_hist32, num_duplicates, ws, s, false);
}

// ----------------------------------------------------------------------------- packed Kronecker ids
// Tables of the digit packing (ByteCount in kron.hpp) for digits 0 .. r-1 of
// a base-2^shift id, g digits per group (bits = g shift bits, r^g <= 255):
// tab[x] = base-r value of the smallest digit-valid group >= x, + 256 if x is
// itself valid; dec[b] = the group whose base-r value is b (b < r^g).
__global__ void pack_tables(uint32_t r, int shift, int g, int bits, uint16_t *tab, uint32_t *dec) {
    const uint32_t dmask = (1u << shift) - 1u;
    for (uint32_t x = threadIdx.x; x < (1u << bits); x += blockDim.x) {
        uint32_t pv = 0, val = 256;
        int i = 0;
        for (; i < g; ++i) {
            const uint32_t d = (x >> (shift * (g - 1 - i))) & dmask;
            if (d >= r) break;
            pv = pv * r + d;
        }
        if (i < g) {  // first invalid digit at i: next prefix, zeros below
            val = pv + 1;
            for (int m = i; m < g; ++m) val *= r;
        } else {
            val |= pv;
        }
        tab[x] = (uint16_t)val;
    }
    uint32_t rg = 1;
    for (int m = 0; m < g; ++m) rg *= r;
    for (uint32_t b = threadIdx.x; b < 256; b += blockDim.x) {
        uint32_t grp = 0, v = b;
        if (b < rg)
            for (int m = 0; m < g; ++m) {
                grp |= (v % r) << (shift * m);
                v /= r;
            }
        dec[b] = grp;
    }
}

// Row starts of all n ids from those of the packed ids: id's row starts where
// the row of the smallest digit-valid id >= id starts (packed rows without an
// id -- byte values >= r^g -- were filled with the next row's start), and
// row_ptr[n] = rpc[nc].
__global__ __launch_bounds__(256) void csr_expand_rows(uint64_t n, uint64_t nc, const uint64_t *rpc,
                                                        uint64_t *row_ptr, const uint16_t *tab, int groups, int bits) {
    // The packing table (at most 2^12 entries) in LDS, and four ids of a
    // 1,024-id chunk per thread: the table lookups stay on the CU and the
    // four row-start reads travel together.
    __shared__ uint16_t s_tab[1 << 12];
    for (uint32_t i = threadIdx.x; i < (1u << bits); i += blockDim.x) s_tab[i] = tab[i];
    __syncthreads();
    const uint64_t gmask = (1ull << bits) - 1;
    for (uint64_t base = (uint64_t)blockIdx.x * 1024; base <= n; base += (uint64_t)gridDim.x * 1024) {
        uint64_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint64_t id = base + 256 * u + threadIdx.x;
            uint64_t p = nc;
            if (id < n) {
                p = 0;
                for (int j = groups - 1; j >= 0; --j) {
                    const uint32_t t = s_tab[(id >> (bits * j)) & gmask];
                    p = (p << 8) | (t & 255u);
                    if (!(t >> 8)) {
                        p <<= 8 * j;
                        break;
                    }
                }
            }
            v[u] = id <= n ? rpc[p] : 0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint64_t id = base + 256 * u + threadIdx.x;
            if (id <= n) row_ptr[id] = v[u];
        }
    }
}

// Degree-0 vertices of the ids that no packed id stands for.
__global__ void hist_add_bin0(uint64_t *hist, uint64_t add) {
    if (threadIdx.x == 0 && blockIdx.x == 0) hist[0] += add;
}

// kron_generate_csr on packed ids (see kron_csr_build).  Returns 1 when the
// configuration does not pack (nothing launched), else the status.
int kron_csr_packed(uint32_t n0, const float *initiator, uint32_t k, uint64_t num_edges, int mode, uint64_t seed,
                    uint32_t graph_id, int id_bytes, void *src, void *dst, uint32_t flags, uint64_t *row_ptr,
                    void *col, uint64_t *degree_hist32, uint64_t *num_duplicates, char *ws, size_t workspace_bytes,
                    const Plan &full, hipStream_t s) {
    if (mode != SFG_KRON_SAMPLE || flags != 0 || (n0 & (n0 - 1)) != 0 || num_edges == 0) return 1;
    SampleTable tab;
    memset(&tab, 0, sizeof(tab));
    if (build_sample_table(n0, initiator, tab) != SFG_OK || tab.nt > 15) return 1;
    uint32_t r = 0;
    for (uint32_t b = 0; b <= tab.nt; ++b) r = std::max<uint32_t>(r, std::max(tab.row[b], tab.col[b]) + 1u);
    if (r >= n0 || r < 2) return 1;
    int shift = 0;
    while ((1u << shift) < n0) ++shift;
    int g = 0;
    for (uint64_t rg = r; rg <= 255 && (g + 1) * shift <= 12; rg *= r) ++g;
    if (g < 1) return 1;
    const int bits = g * shift;
    const int groups = (int)((k + g - 1) / g);
    const int top = (int)k - g * (groups - 1);  // digits of the most significant group
    if (groups > 4) return 1;
    uint64_t rt = 1;
    for (int m = 0; m < top; ++m) rt *= r;
    const uint64_t nc = (rt + 1) << (8 * (groups - 1));  // packed ids below nc, plus the "beyond" row
    uint64_t n = 1;
    for (uint32_t i = 0; i < k; ++i) n *= n0;
    Plan P = make_plan(nc, num_edges, id_bytes, flags, degree_hist32 != nullptr);
    if (P.passes >= full.passes || !P.fused_finish || P.db % 8 != 0 || P.db != 8 * groups) return 1;
    // Layout: the packed CSR's workspace, then its row starts, the two tables.
    const size_t off_rpc = align256(P.total);
    const size_t off_tab = off_rpc + align256((nc + 1) * 8);
    const size_t off_dec = off_tab + align256(((size_t)1 << bits) * 2);
    const size_t need = off_dec + align256(256 * 4);
    if (need > workspace_bytes) return 1;
    uint64_t *rpc = reinterpret_cast<uint64_t *>(ws + off_rpc);
    uint16_t *ptab = reinterpret_cast<uint16_t *>(ws + off_tab);
    uint32_t *dec = reinterpret_cast<uint32_t *>(ws + off_dec);
    { ProfScope _ps("fill", s); pack_tables<<<1, 256, 0, s>>>(r, shift, g, bits, ptab, dec); }
    ByteCount bc{};
    bc.hist = reinterpret_cast<uint64_t *>(ws + P.off_ghist);
    bc.rows = P.passes;
    bc.row_mod = P.passes;
    bc.dst_row = 0;
    bc.dst_bytes = P.dpasses;
    bc.src_row = P.dpasses;
    bc.src_bytes = P.passes - P.dpasses;
    bc.key_shift = P.db;
    if (P.key_bytes == 8)
        bc.keys = reinterpret_cast<uint64_t *>(ws + first_input_offset(P));
    else
        bc.keys32 = reinterpret_cast<uint32_t *>(ws + first_input_offset(P));
    bc.pack_groups = groups;
    bc.pack_bits = bits;
    bc.pack_base = r;
    bc.pack_tab = ptab;
    clear_csr(P, rpc, degree_hist32, num_duplicates, ws, s);
    bool counted = false;
    int rc = kron_generate_counted(n0, initiator, k, num_edges, 0, num_edges, mode, seed, graph_id, id_bytes, src, dst,
                                   s, &bc, &counted);
    if (rc != SFG_OK) return rc;
    if (!counted)  // the sampler wrote the ids only: build from them unpacked
        return csr_run(full, src, dst, id_bytes, row_ptr, col, degree_hist32, num_duplicates, ws, s, false);
    const Unpack up{dec, groups, bits};
    rc = csr_run(P, src, dst, id_bytes, rpc, col, degree_hist32, num_duplicates, ws, s, true, true, &up);
    if (rc != SFG_OK) return rc;
    {
        ProfScope _ps("csr_rowfill", s);
        csr_expand_rows<<<fill_grid(n + 1), 256, 0, s>>>(n, nc, rpc, row_ptr, ptab, groups, bits);
    }
    if (degree_hist32) { ProfScope _ps("fill", s); hist_add_bin0<<<1, 64, 0, s>>>(degree_hist32, n - nc); }
    return check_launch("kron_generate_csr");
}

// Kronecker edges straight into their CSR.  The key's digits are whole bytes
// of the ids when the destination field is a whole number of bytes: digit p
// is destination byte p below the field's dpasses bytes and source byte
// p - dpasses above (symmetrized: byte p mod dpasses of both ends, the two
// orientations of an edge together).  The sampler counts those bytes as it
// writes the ids, which replaces the histogram pass's read of the edge list.
int kron_csr_build(uint32_t n0, const float *initiator, uint32_t k, uint64_t num_edges, int mode, uint64_t seed,
                   uint32_t graph_id, int id_bytes, void *src, void *dst, uint32_t flags, uint64_t *row_ptr,
                   void *col, uint64_t *degree_hist32, uint64_t *num_duplicates, void *workspace,
                   size_t workspace_bytes, hipStream_t s) {
    if (n0 < 2) return fail(SFG_EINVAL, "kron_generate_csr: n0 must be >= 2 (got %u)", n0);
    if (k == 0) return fail(SFG_EINVAL, "kron_generate_csr: k must be >= 1");
    uint64_t n = 1;
    for (uint32_t i = 0; i < k; ++i) {
        if (n > (1ull << 32) / n0) return fail(SFG_ERANGE, "kron_generate_csr: %u^%u vertices exceed 2^32", n0, k);
        n *= n0;
    }
    Plan P;
    int rc = csr_check(n, num_edges, src, dst, id_bytes, flags, row_ptr, col, degree_hist32, workspace,
                       workspace_bytes, P);
    if (rc != SFG_OK) return rc;
    // The generator's own checks, with no edge to write: nothing is launched
    // unless every argument is valid.
    rc = kron_generate_counted(n0, initiator, k, num_edges, 0, 0, mode, seed, graph_id, id_bytes, src, dst, s, nullptr,
                               nullptr);
    if (rc != SFG_OK) return rc;
    char *ws = static_cast<char *>(workspace);
    // A zero-padded initiator (its last rows and columns zero, so the ids'
    // digits stay below r < n0): the sort runs on packed ids, g digits per
    // byte, which shortens the keys by whole passes; the last pass unpacks
    // the columns and the row starts of all n ids are expanded from those of
    // the packed ids.  Outputs are the same as without packing.
    rc = kron_csr_packed(n0, initiator, k, num_edges, mode, seed, graph_id, id_bytes, src, dst, flags, row_ptr, col,
                         degree_hist32, num_duplicates, ws, workspace_bytes, P, s);
    if (rc != 1) return rc;  // done (SFG_OK) or failed; 1 = not applicable
    ByteCount bc{};
    const bool bytes = P.db % 8 == 0 && P.N > 0;
    if (bytes) {
        bc.hist = reinterpret_cast<uint64_t *>(ws + P.off_ghist);
        bc.rows = P.passes;
        if (P.sym) {
            bc.row_mod = P.dpasses;
            bc.dst_row = bc.src_row = 0;
            bc.dst_bytes = bc.src_bytes = P.dpasses;
        } else {
            bc.row_mod = P.passes;
            bc.dst_row = 0;
            bc.dst_bytes = P.dpasses;
            bc.src_row = P.dpasses;
            bc.src_bytes = P.passes - P.dpasses;
        }
        clear_csr(P, row_ptr, degree_hist32, num_duplicates, ws, s);
        // 8-byte keys: the sampler writes them too, and the first pass
        // reads them instead of the two id arrays.
        if (P.key_bytes == 8) {
            bc.keys = reinterpret_cast<uint64_t *>(ws + first_input_offset(P));
            bc.key_shift = P.db;
            bc.key_sym = P.sym;
        }
    }
    bool counted = false;
    rc = kron_generate_counted(n0, initiator, k, num_edges, 0, num_edges, mode, seed, graph_id, id_bytes, src, dst, s,
                               bytes ? &bc : nullptr, &counted);
    if (rc != SFG_OK) return rc;
    return csr_run(P, src, dst, id_bytes, row_ptr, col, degree_hist32, num_duplicates, ws, s, counted,
                   counted && bc.keys != nullptr);
}

}  // namespace sfg

namespace sfg {

namespace {
// The tables of power.hpp, a workgroup per row of a digit's seed: blocks
// [0, c.n[0]) and the next c.n[1] the counting rows, then those for walking.
// Every workgroup derives the seed's own rows from its bits first.
__global__ __launch_bounds__(64) void power_tables(PowerSeed q, PowerDigits c, PowerDigits w, PowerTables *t) {
    __shared__ uint8_t s_list[kPowerMaxN0 * kPowerMaxN0];
    __shared__ uint32_t s_start[kPowerMaxN0 + 1];
    const uint32_t n0 = q.n0, tid = threadIdx.x;
    auto cell = [&](uint32_t a, uint32_t b) { return (q.mask[(a * n0 + b) / 32] >> ((a * n0 + b) % 32)) & 1u; };
    uint32_t deg0 = 0;
    if (tid < n0)
        for (uint32_t y = 0; y < n0; ++y) deg0 += cell(tid, y);
    uint32_t sum = deg0;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_up(sum, off, 64);
        if (tid >= (uint32_t)off) sum += o;
    }
    s_start[tid + 1] = sum;
    if (tid == 0) s_start[0] = 0;
    if (tid < n0) {
        uint32_t at = sum - deg0;
        for (uint32_t y = 0; y < n0; ++y)
            if (cell(tid, y)) s_list[at++] = (uint8_t)y;
    }
    __syncthreads();
    uint32_t x = blockIdx.x;
    const bool counting = x < c.n[0] + c.n[1];
    if (!counting) x -= c.n[0] + c.n[1];
    const PowerDigits &p = counting ? c : w;
    const uint32_t v = x < p.n[0] ? 0 : 1, n = p.n[v], levels = p.levels[v];
    if (v) x -= p.n[0];
    // Entries of row x and of the rows below it, most significant level first.
    uint32_t start = 0, deg = 1, place = n, entries = 1;
    for (uint32_t l = 0; l < levels; ++l) entries *= q.e0;
    for (uint32_t l = 0, xx = x, below = entries; l < levels; ++l) {
        place /= n0;
        below /= q.e0;
        const uint32_t dgt = xx / place;
        xx -= dgt * place;
        start += deg * s_start[dgt] * below;
        deg *= s_start[dgt + 1] - s_start[dgt];
    }
    if (counting) {
        uint8_t *rank = t->count.rank + (v ? p.n[0] * p.n[0] : 0) + x * n;
        for (uint32_t y = tid; y < n; y += 64) {
            uint32_t r = 0;
            bool in = true;
            uint32_t pl = n, xx = x, yy = y;
            for (uint32_t l = 0; l < levels; ++l) {
                pl /= n0;
                const uint32_t a = xx / pl, b = yy / pl;
                xx -= a * pl;
                yy -= b * pl;
                uint32_t below = 0;
                for (uint32_t z = 0; z < b; ++z) below += cell(a, z);
                r = r * (s_start[a + 1] - s_start[a]) + (in ? below : 0);
                in = in && cell(a, b);
            }
            rank[y] = (uint8_t)(r | (in ? 0x80u : 0u));
        }
        if (tid == 0) {
            t->count.start[v][x] = (uint16_t)start;
            if (x + 1 == n) t->count.start[v][n] = (uint16_t)entries;
        }
    } else {
        for (uint32_t i = tid; i < deg; i += 64) {
            uint32_t y = 0, ii = i, xx = x, pl = 1;
            for (uint32_t l = 0; l < levels; ++l) {  // least significant level first
                const uint32_t a = xx % n0, s = s_start[a], d = s_start[a + 1] - s;
                y += s_list[s + ii % d] * pl;
                ii /= d;
                xx /= n0;
                pl *= n0;
            }
            t->list[v][start + i] = (uint16_t)y;
            t->rowof[v][start + i] = (uint16_t)x;
        }
        if (tid == 0) {
            t->start[v][x] = (uint16_t)start;
            t->degmagic[v][x] = deg ? 0xFFFFFFFFu / deg : 0;
            if (x + 1 == n) t->start[v][n] = (uint16_t)entries;
        }
    }
}
}  // namespace

size_t csr_xor_workspace_bytes(uint64_t n, uint64_t num_random, uint64_t num_power) {
    return make_plan(n, num_random, 8, 0, false, true, num_power).total;
}

int csr_xor_begin(uint64_t n, uint64_t num_random, Power *power, const PowerSeed &seed, uint64_t *row_ptr, void *workspace,
                  size_t workspace_bytes, hipStream_t s, XorKeys *keys) {
    if (n > (1ull << 31)) return fail(SFG_ERANGE, "xor: n above 2^31 does not fit the tagged key");
    if (!device_error_word()) return fail(SFG_EDEVICE, "xor: no device");
    const Plan P = make_plan(n, num_random, 8, 0, false, true, power->entries);
    if (workspace_bytes < P.total)
        return fail(SFG_ENOSPACE, "xor: workspace has %zu bytes, needs %zu", workspace_bytes, P.total);
    char *ws = static_cast<char *>(workspace);
    clear_csr(P, row_ptr, nullptr, nullptr, ws, s);
    PowerTables *t = reinterpret_cast<PowerTables *>(ws + P.off_tables);
    power->tables = t;
    { ProfScope _ps("fill", s); power_tables<<<power->c.n[0] + power->c.n[1] + power->w.n[0] + power->w.n[1], 64, 0, s>>>(seed, power->c, power->w, t); }
    keys->keys = ws + first_input_offset(P);
    keys->hist = reinterpret_cast<uint64_t *>(ws + P.off_ghist);
    keys->key_bytes = P.key_bytes;
    keys->shift = P.db;
    keys->passes = P.passes;
    return SFG_OK;
}

int csr_xor_finish(uint64_t n, uint64_t num_random, const Power &power, int id_bytes, uint64_t *row_ptr, void *col,
                   void *workspace, hipStream_t s) {
    const Plan P = make_plan(n, num_random, 8, 0, false, true, power.entries);
    char *ws = static_cast<char *>(workspace);
    if (P.key_bytes == 4) {
        if (id_bytes == 4)
            return run_csr<int32_t, uint32_t>(P, nullptr, nullptr, row_ptr, col, nullptr, nullptr, ws, s, true, true, nullptr, &power);
        return run_csr<int64_t, uint32_t>(P, nullptr, nullptr, row_ptr, col, nullptr, nullptr, ws, s, true, true, nullptr, &power);
    }
    if (id_bytes == 4)
        return run_csr<int32_t, uint64_t>(P, nullptr, nullptr, row_ptr, col, nullptr, nullptr, ws, s, true, true, nullptr, &power);
    return run_csr<int64_t, uint64_t>(P, nullptr, nullptr, row_ptr, col, nullptr, nullptr, ws, s, true, true, nullptr, &power);
}

}  // namespace sfg

extern "C" int kron_generate_csr(uint32_t n0, const float *initiator, uint32_t k, uint64_t num_edges, int mode,
                                 uint64_t seed, uint32_t graph_id, int id_bytes, void *src, void *dst, uint32_t flags,
                                 uint64_t *row_ptr, void *col, uint64_t *degree_hist32, uint64_t *num_duplicates,
                                 void *workspace, size_t workspace_bytes, void *stream) {
    return kron_csr_build(n0, initiator, k, num_edges, mode, seed, graph_id, id_bytes, src, dst, flags, row_ptr, col,
                          degree_hist32, num_duplicates, workspace, workspace_bytes, as_stream(stream));
}

extern "C" int edges_to_csr(uint64_t n, uint64_t num_edges, const void *src, const void *dst, int id_bytes,
                            uint32_t flags, uint64_t *row_ptr, void *col, uint64_t *degree_hist32,
                            uint64_t *num_duplicates, void *workspace, size_t workspace_bytes, void *stream) {
    return csr_build(n, num_edges, src, dst, id_bytes, flags, row_ptr, col, degree_hist32, num_duplicates, workspace,
                     workspace_bytes, as_stream(stream), nullptr);
}

// --------------------------------------------------------------------------- no-allocation variant
// edges_to_csr for callers that cannot allocate (code under stream capture,
// serving loops, harnesses without hipMalloc): the workspace is a file-scope
// device array of kNoAllocScratch bytes instead of a caller buffer.  Every
// device holds its own copy at its own address, looked up once per device;
// host code passes that address, never the array's name, to the kernels.
namespace sfg {
namespace {
constexpr size_t kNoAllocScratch = 64ull << 20;
__device__ __align__(256) unsigned char scratch[kNoAllocScratch];

char *noalloc_scratch() {
    static constexpr int kMaxDevs = 64;
    static char *addr[kMaxDevs] = {nullptr};
    static std::mutex mu;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevs) return nullptr;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
        addr[dev] = static_cast<char *>(ptr);
    }
    return addr[dev];
}
}  // namespace
}  // namespace sfg

extern "C" size_t edges_to_csr_noalloc_max_bytes(void) { return sfg::kNoAllocScratch; }

extern "C" int edges_to_csr_noalloc(uint64_t n, uint64_t num_edges, const void *src, const void *dst, int id_bytes,
                                    uint32_t flags, uint64_t *row_ptr, void *col, uint64_t *degree_hist32,
                                    uint64_t *num_duplicates, void *stream) {
    if (n > 0 && (id_bytes == 4 || id_bytes == 8)) {
        const size_t need = sfg::csr_workspace_bytes(n, num_edges, id_bytes, flags);
        if (need > sfg::kNoAllocScratch)
            return fail(SFG_ERANGE,
                        "edges_to_csr_noalloc: %llu vertices and %llu edges need %zu scratch bytes, more than the "
                        "%zu of the static scratch array",
                        (unsigned long long)n, (unsigned long long)num_edges, need, sfg::kNoAllocScratch);
    }
    char *ws = sfg::noalloc_scratch();
    if (!ws) return fail(SFG_EDEVICE, "edges_to_csr_noalloc: scratch address lookup failed");
    return csr_build(n, num_edges, src, dst, id_bytes, flags, row_ptr, col, degree_hist32, num_duplicates, ws,
                     sfg::kNoAllocScratch, as_stream(stream), nullptr);
}
