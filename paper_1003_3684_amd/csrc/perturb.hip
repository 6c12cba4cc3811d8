// Randomized PK by temporary seed modification (PK section, randomization):
// at every expansion a meta-edge is replaced by the edges of its own
// perturbed copy of the seed (absent cells added with probability p_add,
// present cells deleted with probability p_del; draws keyed by the
// meta-edge's iteration and coordinates).
//
// The paper's processors expand meta-edges depth first.  Here the expansion
// is level-synchronous: per iteration every meta-edge draws its perturbed cell
// mask, a scan of the fan-outs of granules of meta-edges gives each granule its
// output range, and a second sweep writes the children in cell order.  That
// order is the depth-first order of the paper's stack, so the edge list is
// the same, entry for entry.  The fan-out varies per meta-edge, which is why
// the scan is needed.  The level sizes stay on the device: every level's
// kernels read the size that the scan before them left, a level above the
// capacity stops the ones after it, and the host reads all sizes once, at the
// end.  (The scan is a launch of its own and not a look-back, so that calls on
// several streams may overlap.)
#include <string.h>

#include <algorithm>

#include "common.hpp"

namespace sfg {
namespace {

constexpr uint32_t TAG_PERTURB = 7;
constexpr int kPtThreads = 256;
constexpr int kPtRounds = 4;                              // meta-edges per thread and granule
constexpr uint64_t kGranule = kPtThreads * kPtRounds;     // meta-edges
constexpr uint32_t kPtLevels = 33;                        // n0^k <= 2^32: sizes of levels 1 .. k
constexpr uint64_t kPtOverflow = ~0ull;                   // size of a level after one that was too large

struct PtArgs {
    uint64_t adj;            // seed cells as bits (n0 <= 8)
    uint64_t flippable;      // cells whose probability is not 0
    uint32_t n0, cells;
    uint32_t inv;            // cell / n0 = cell inv >> 10, for cells below 64
    uint32_t key0, key1, tagword;
    uint32_t add_m1, del_m1;  // a cell flips where its word is at most this
    uint64_t capacity;
};

// The perturbed cell mask of meta-edge (iteration it, row, col): the seed's
// cells, each flipped (added or deleted) by its own word.
template <typename MaskT>
__device__ __forceinline__ MaskT perturbed_mask(const PtArgs &a, uint32_t it, uint32_t row, uint32_t col) {
    MaskT flips = 0;
    for (uint32_t b = 0; b * 4 < a.cells; ++b) {
        const Block4 r = philox(row, col, it | (b << 8), a.tagword, a.key0, a.key1);
        const uint32_t w[4] = {r.w0, r.w1, r.w2, r.w3}, seed = (uint32_t)(a.adj >> (4 * b));
        uint32_t four = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) four |= (w[i] <= ((seed >> i) & 1u ? a.del_m1 : a.add_m1) ? 1u : 0u) << i;
        flips |= (MaskT)four << (4 * b);
    }
    return (MaskT)a.adj ^ (flips & (MaskT)a.flippable);  // (words past the last cell: not flippable)
}

// Level 1: the seed's own edges, row-major (the stack's order), to the
// caller's arrays if there is no other level.
template <typename OutT>
__global__ __launch_bounds__(64) void pt_seed(PtArgs a, OutT *row, OutT *col, uint64_t *sizes, uint64_t *num_edges) {
    const uint32_t c = threadIdx.x;
    if ((a.adj >> c) & 1u) {
        const uint32_t at = (uint32_t)__popcll(a.adj & ((1ull << c) - 1));
        row[at] = (OutT)(c / a.n0);
        col[at] = (OutT)(c % a.n0);
    }
    if (c == 0) {
        sizes[1] = (uint64_t)__popcll(a.adj);
        if (num_edges) *num_edges = sizes[1];
    }
}

// The size of level it, 0 if it or one before it was too large.
__device__ __forceinline__ uint64_t level_size(const PtArgs &a, const uint64_t *sizes, uint32_t it) {
    const uint64_t n = sizes[it];
    return n <= a.capacity ? n : 0;
}

// Masks of level it and the fan-outs of its granules.  Bound by the
// generator's instructions (seven Philox blocks per meta-edge at n0 = 5).  The
// masks are kept, 4 bytes per meta-edge up to 32 cells: a level took a fan-out
// pass, three scan launches over 4-byte fan-outs and 8-byte offsets, and an
// expansion that drew the masks again.  For the 2.1e8 edges of seven expansions
// of an 11-edge seed that was 355 + 511 + 910 us and seven waits of the host, now
// 303 (masks) + 60 (scans) + 587 (expansion: 1.9 GB, 3.3 TB/s) and one.
template <typename MaskT>
__global__ __launch_bounds__(kPtThreads) void pt_masks(PtArgs a, uint32_t it, const uint64_t *sizes, const uint32_t *row,
                                                       const uint32_t *col, MaskT *masks, uint64_t *sums) {
    __shared__ uint32_t s_w[kPtThreads / 64];
    const uint64_t count = level_size(a, sizes, it);
    for (uint64_t g = blockIdx.x; g * kGranule < count; g += gridDim.x) {
        uint32_t fan = 0;
#pragma unroll
        for (int q = 0; q < kPtRounds; ++q) {
            const uint64_t j = g * kGranule + q * kPtThreads + threadIdx.x;
            if (j < count) {
                const MaskT m = perturbed_mask<MaskT>(a, it, row[j], col[j]);
                masks[j] = m;
                fan += (uint32_t)__popcll((uint64_t)m);
            }
        }
        for (int off = 32; off > 0; off >>= 1) fan += __shfl_xor(fan, off, 64);
        if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = fan;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint64_t t = 0;
            for (int w = 0; w < kPtThreads / 64; ++w) t += s_w[w];
            sums[g] = t;
        }
        __syncthreads();
    }
}

// Exclusive scan of the granules' fan-outs, in place; the size of level it + 1.
__global__ __launch_bounds__(1024) void pt_scan(PtArgs a, uint32_t it, uint64_t *sizes, uint64_t *sums, uint64_t *num_edges) {
    __shared__ uint64_t s[1024];
    const uint64_t count = level_size(a, sizes, it), nb = (count + kGranule - 1) / kGranule;
    const uint64_t per = (nb + 1023) / 1024;
    const uint64_t lo = min((uint64_t)threadIdx.x * per, nb), hi = min(lo + per, nb);
    uint64_t x = 0;
    for (uint64_t i = lo; i < hi; ++i) x += sums[i];
    s[threadIdx.x] = x;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const uint64_t y = threadIdx.x >= (unsigned)off ? s[threadIdx.x - off] : 0;
        __syncthreads();
        s[threadIdx.x] += y;
        __syncthreads();
    }
    uint64_t run = s[threadIdx.x] - x;  // exclusive prefix of this thread's range
    for (uint64_t i = lo; i < hi; ++i) {
        const uint64_t v = sums[i];
        sums[i] = run;
        run += v;
    }
    if (threadIdx.x == 1023) {
        const uint64_t total = sizes[it] <= a.capacity ? s[1023] : kPtOverflow;
        sizes[it + 1] = total;
        if (num_edges && total <= a.capacity) *num_edges = total;
    }
}

// Children of every meta-edge, in cell order.  A granule's output range is
// known; in it, kPtThreads meta-edges at a time are scanned (the fan-outs of
// all rounds at once, 16 bits each: at most 256 x 64), their children are put
// into LDS in order as (parent, cell) and written out coalesced.
template <typename MaskT, typename OutT>
__global__ __launch_bounds__(kPtThreads) void pt_expand(PtArgs a, uint32_t it, const uint64_t *sizes, const uint32_t *row,
                                                        const uint32_t *col, const MaskT *masks, const uint64_t *sums,
                                                        OutT *nrow, OutT *ncol) {
    __shared__ uint16_t s_child[kPtThreads * sizeof(MaskT) * 8];  // parent << 6 | cell
    __shared__ uint32_t s_row[kPtThreads], s_col[kPtThreads];
    __shared__ uint64_t s_w[kPtThreads / 64];
    static_assert(kPtRounds == 4 && kPtThreads * 64 < (1 << 16), "four 16-bit fan-out sums, 14-bit children");
    const uint64_t count = level_size(a, sizes, it);
    if (sizes[it + 1] > a.capacity) return;
    const int tid = threadIdx.x;
    const uint32_t lane = tid & 63;
    for (uint64_t g = blockIdx.x; g * kGranule < count; g += gridDim.x) {
        MaskT m[kPtRounds];
        uint64_t fan = 0;
#pragma unroll
        for (int q = 0; q < kPtRounds; ++q) {
            const uint64_t j = g * kGranule + q * kPtThreads + tid;
            m[q] = j < count ? masks[j] : (MaskT)0;
            fan |= (uint64_t)__popcll((uint64_t)m[q]) << (16 * q);
        }
        uint64_t x = fan;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint64_t y = __shfl_up(x, off, 64);
            if (lane >= (uint32_t)off) x += y;
        }
        if (lane == 63) s_w[tid >> 6] = x;
        __syncthreads();
        uint64_t all = 0;
        x -= fan;
#pragma unroll
        for (int w = 0; w < kPtThreads / 64; ++w) {
            if (w < (tid >> 6)) x += s_w[w];
            all += s_w[w];
        }
        uint64_t out = sums[g];
#pragma unroll
        for (int q = 0; q < kPtRounds; ++q) {
            const uint64_t j = g * kGranule + q * kPtThreads + tid;
            const uint32_t n = (uint32_t)(all >> (16 * q)) & 0xFFFFu;
            uint32_t o = (uint32_t)(x >> (16 * q)) & 0xFFFFu;
            if (j < count) {
                s_row[tid] = row[j] * a.n0;
                s_col[tid] = col[j] * a.n0;
            }
            for (MaskT left = m[q]; left; left &= left - 1)
                s_child[o++] = (uint16_t)(tid << 6 | (sizeof(MaskT) == 4 ? __builtin_ctz((uint32_t)left) : __builtin_ctzll((uint64_t)left)));
            __syncthreads();
            for (uint32_t i = tid; i < n; i += kPtThreads) {
                const uint32_t child = s_child[i], parent = child >> 6, cell = child & 63u, cr = cell * a.inv >> 10;
                nrow[out + i] = (OutT)(s_row[parent] + cr);
                ncol[out + i] = (OutT)(s_col[parent] + cell - cr * a.n0);
            }
            out += n;
            __syncthreads();
        }
    }
}

// Workgroups for a level of at most `items` meta-edges.
int grid_of(uint64_t items) {
    return (int)std::max<uint64_t>(1, std::min<uint64_t>((items + kGranule - 1) / kGranule, (uint64_t)device_cu_count() * 8));
}

struct PtPlan {
    size_t off_r0, off_c0, off_r1, off_c1, off_masks, off_sums, off_sizes, total;
};

template <typename MaskT>
void launch_level(const PtArgs &a, uint32_t it, int g, uint64_t *sizes, const uint32_t *row, const uint32_t *col, MaskT *masks,
                  uint64_t *sums, bool last, int id_bytes, void *nrow, void *ncol, uint64_t *num_edges, hipStream_t s) {
    pt_masks<MaskT><<<g, kPtThreads, 0, s>>>(a, it, sizes, row, col, masks, sums);
    pt_scan<<<1, 1024, 0, s>>>(a, it, sizes, sums, last ? num_edges : nullptr);
    if (!last)
        pt_expand<MaskT, uint32_t><<<g, kPtThreads, 0, s>>>(a, it, sizes, row, col, masks, sums, static_cast<uint32_t *>(nrow),
                                                            static_cast<uint32_t *>(ncol));
    else if (id_bytes == 4)
        pt_expand<MaskT, int32_t><<<g, kPtThreads, 0, s>>>(a, it, sizes, row, col, masks, sums, static_cast<int32_t *>(nrow),
                                                           static_cast<int32_t *>(ncol));
    else
        pt_expand<MaskT, int64_t><<<g, kPtThreads, 0, s>>>(a, it, sizes, row, col, masks, sums, static_cast<int64_t *>(nrow),
                                                           static_cast<int64_t *>(ncol));
}

PtPlan pt_plan(uint64_t capacity) {
    PtPlan p;
    size_t o = 0;
    auto take = [&](size_t b) {
        size_t r = o;
        o += align256(b);
        return r;
    };
    p.off_r0 = take(capacity * 4);
    p.off_c0 = take(capacity * 4);
    p.off_r1 = take(capacity * 4);
    p.off_c1 = take(capacity * 4);
    p.off_masks = take(capacity * 8);
    p.off_sums = take(((capacity + kGranule - 1) / kGranule + 1) * 8);
    p.off_sizes = take(kPtLevels * 8);
    p.total = o;
    return p;
}

}  // namespace
}  // namespace sfg

using namespace sfg;

extern "C" size_t kron_perturbed_workspace_bytes(uint64_t capacity) { return pt_plan(std::max<uint64_t>(capacity, 1)).total; }

extern "C" int kron_perturbed(uint32_t n0, const float *seed_matrix, uint32_t k, double p_add, double p_del,
                              uint64_t seed, uint32_t graph_id, int id_bytes, uint64_t capacity, void *src, void *dst,
                              uint64_t *num_edges, void *workspace, size_t workspace_bytes, void *stream) {
    if (n0 < 2 || n0 > 8) return fail(SFG_EINVAL, "kron_perturbed: n0 must be in [2, 8]");
    if (k == 0) return fail(SFG_EINVAL, "kron_perturbed: k must be >= 1");
    if (!seed_matrix) return fail(SFG_EINVAL, "kron_perturbed: NULL seed matrix");
    if (!(p_add >= 0.0 && p_add <= 1.0) || !(p_del >= 0.0 && p_del <= 1.0))
        return fail(SFG_EINVAL, "kron_perturbed: probabilities must be in [0, 1]");
    if (id_bytes != 4 && id_bytes != 8) return fail(SFG_EINVAL, "kron_perturbed: id_bytes must be 4 or 8");
    if (graph_id >= (1u << 24)) return fail(SFG_EINVAL, "kron_perturbed: graph_id must be < 2^24");
    if (k > 255) return fail(SFG_ERANGE, "kron_perturbed: k above 255");
    uint64_t n = 1;
    for (uint32_t l = 0; l < k; ++l) {
        if (n > (1ull << 32) / n0) return fail(SFG_ERANGE, "kron_perturbed: n0^k above 2^32");
        n *= n0;
    }
    if (id_bytes == 4 && n - 1 > 0x7FFFFFFFull) return fail(SFG_ERANGE, "kron_perturbed: ids do not fit int32");
    PtArgs a;
    memset(&a, 0, sizeof(a));
    a.n0 = n0;
    a.cells = n0 * n0;
    uint32_t e0 = 0;
    for (uint32_t c = 0; c < a.cells; ++c) {
        if (!(seed_matrix[c] >= 0.0f) || seed_matrix[c] > 3.0e38f)
            return fail(SFG_EINVAL, "kron_perturbed: bad seed entry %u", c);
        if (seed_matrix[c] != 0.0f) {
            a.adj |= 1ull << c;
            ++e0;
        }
    }
    if (e0 == 0) return fail(SFG_EINVAL, "kron_perturbed: the seed graph has no edge");
    if (!num_edges || (capacity > 0 && (!src || !dst))) return fail(SFG_EINVAL, "kron_perturbed: NULL output");
    const PtPlan P = pt_plan(std::max<uint64_t>(capacity, 1));
    if (!workspace) return fail(SFG_EINVAL, "kron_perturbed: workspace is NULL");
    if (workspace_bytes < P.total)
        return fail(SFG_ENOSPACE, "kron_perturbed: workspace has %zu bytes, needs %zu", workspace_bytes, P.total);
    if (capacity < e0) return fail(SFG_ENOSPACE, "kron_perturbed: capacity below the %u seed edges", e0);
    // floor(p 2^32) in binary64: a cell flips where its 32-bit word is below it.
    const uint64_t thr_add = (uint64_t)(p_add * 4294967296.0), thr_del = (uint64_t)(p_del * 4294967296.0);
    a.add_m1 = (uint32_t)(thr_add - 1);
    a.del_m1 = (uint32_t)(thr_del - 1);
    const uint64_t all_cells = a.cells == 64 ? ~0ull : (1ull << a.cells) - 1;
    a.flippable = (thr_add ? all_cells & ~a.adj : 0) | (thr_del ? a.adj : 0);
    a.inv = (1024 + n0 - 1) / n0;
    a.capacity = capacity;
    a.key0 = (uint32_t)seed;
    a.key1 = (uint32_t)(seed >> 32);
    a.tagword = TAG_PERTURB | (graph_id << 8);
    hipStream_t s = as_stream(stream);
    char *ws = static_cast<char *>(workspace);
    uint32_t *r0 = reinterpret_cast<uint32_t *>(ws + P.off_r0), *c0 = reinterpret_cast<uint32_t *>(ws + P.off_c0);
    uint32_t *r1 = reinterpret_cast<uint32_t *>(ws + P.off_r1), *c1 = reinterpret_cast<uint32_t *>(ws + P.off_c1);
    void *masks = ws + P.off_masks;
    uint64_t *sums = reinterpret_cast<uint64_t *>(ws + P.off_sums), *sizes = reinterpret_cast<uint64_t *>(ws + P.off_sizes);

    // Level 1, then the expansions it -> it + 1 for it = 1 .. k-1; the last
    // level goes to the caller's arrays.
    {
        ProfScope _ps("perturb_expand", s);
        if (k > 1)
            pt_seed<uint32_t><<<1, 64, 0, s>>>(a, r0, c0, sizes, nullptr);
        else if (id_bytes == 4)
            pt_seed<int32_t><<<1, 64, 0, s>>>(a, static_cast<int32_t *>(src), static_cast<int32_t *>(dst), sizes, num_edges);
        else
            pt_seed<int64_t><<<1, 64, 0, s>>>(a, static_cast<int64_t *>(src), static_cast<int64_t *>(dst), sizes, num_edges);
    }
    uint64_t bound = e0;  // of the level's size
    for (uint32_t it = 1; it < k; ++it) {
        const int g = grid_of(bound);
        const bool last = it + 1 == k;
        ProfScope _ps("perturb_expand", s);
        if (a.cells <= 32)
            launch_level(a, it, g, sizes, r0, c0, static_cast<uint32_t *>(masks), sums, last, id_bytes, last ? src : r1,
                         last ? dst : c1, num_edges, s);
        else
            launch_level(a, it, g, sizes, r0, c0, static_cast<uint64_t *>(masks), sums, last, id_bytes, last ? src : r1,
                         last ? dst : c1, num_edges, s);
        std::swap(r0, r1);
        std::swap(c0, c1);
        bound = std::min(capacity, bound * a.cells);  // (capacity below 2^58: its arrays are bytes)
    }
    uint64_t found[kPtLevels];
    if (hipMemcpyAsync(found, sizes, (k + 1) * 8, hipMemcpyDeviceToHost, s) != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
        return fail(SFG_EDEVICE, "kron_perturbed: %s", hipGetErrorString(hipGetLastError()));
    for (uint32_t it = 2; it <= k; ++it)
        if (found[it] > capacity)
            return fail(SFG_ENOSPACE, "kron_perturbed: iteration %u has %llu edges, capacity is %llu", it,
                        (unsigned long long)found[it], (unsigned long long)capacity);
    return check_launch("kron_perturbed");
}
