// Graph statistics: the 32-bin degree histogram, the tail exponent of the
// degree distribution and a wedge-closure sample, for one graph or for every
// graph of a batch whose edge lists share one vertex space (graph g owns
// vertices [v0, v1)).
//
// The paper characterises its graphs by their degree distributions and fitted
// power-law exponents (Results, Fig. 3; a finite mean degree implies
// gamma > 2).  The exponent here is the discrete maximum-likelihood
// approximation of Clauset, Shalizi & Newman (SIAM Review 2009):
//   gamma = 1 + N_t / sum_{d >= d_min} ln(d / (d_min - 1/2)),
// over vertices of degree >= d_min = 2 ceil(2E / n), computed in binary64.
// The summation order is fixed by the graph's own vertex numbering (chunks of
// 4096 vertices, a fixed tree inside each chunk and across chunks), so a graph
// gets the same bits alone or inside a batch, on every run and device.
// Wedges are sampled on the simple undirected graph (symmetrized, no
// self-loops, no repeats): centre v with probability proportional to
// C(d_v, 2), then two distinct neighbours; the wedge is closed when they are
// adjacent.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "common.hpp"
#include "stats.hpp"

namespace sfg {
namespace {

constexpr int kChunk = 4096;  // vertices per statistics chunk
constexpr int kChunkThreads = 256;
constexpr int kPer = kChunk / kChunkThreads;

__device__ __forceinline__ int log2_bin(uint64_t d) {
    if (d == 0) return 0;
    const int b = 64 - __clzll(d);  // floor(log2 d) + 1
    return b > 31 ? 31 : b;
}

// The graph owning statistics chunk c (binary search over chunk0).
__device__ __forceinline__ uint32_t graph_of_chunk(const StatGraph *G, uint32_t count, uint64_t c) {
    uint32_t lo = 0, hi = count;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) / 2;
        if (G[mid].chunk0 <= c)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// Row starts v0 .. v0 + kChunk (those up to `last`) into LDS, coalesced.  A
// thread then takes kPer consecutive vertices; one pad slot per kPer spreads
// their reads over the banks.
constexpr int kRowSlots = kChunk + kChunk / kPer + 1;
__device__ __forceinline__ int row_slot(int i) { return i + i / kPer; }
__device__ __forceinline__ void load_rows(const uint64_t *rows, uint64_t v0, uint64_t last, uint64_t *s_row /*[kRowSlots]*/) {
    uint64_t x[kPer + 1];
#pragma unroll
    for (int j = 0; j < kPer; ++j) x[j] = rows[min(v0 + j * kChunkThreads + threadIdx.x, last)];
    x[kPer] = rows[min(v0 + kChunk, last)];
#pragma unroll
    for (int j = 0; j < kPer; ++j) s_row[row_slot(j * kChunkThreads + (int)threadIdx.x)] = x[j];
    if (threadIdx.x == 0) s_row[row_slot(kChunk)] = x[kPer];
}

__device__ __forceinline__ uint64_t pairs_of(uint64_t d) { return d >= 2 ? d * (d - 1) / 2 : 0; }

struct ChunkArgs {
    const StatGraph *G;
    uint32_t count;
    uint64_t total;       // statistics chunks
    const uint64_t *raw;  // multigraph row starts
    uint64_t *hist;
    double *psum;
    uint64_t *pcnt;
    uint32_t grid;        // workgroups of the statistics; the others sum the wedges of one chunk each
    const uint64_t *rp;   // simple row starts of the nv vertices
    uint64_t nv, *csum;
};

// The first `grid` workgroups walk the statistics chunks (persistent: a grid
// smaller than the chunk count takes chunks blockIdx.x, blockIdx.x + grid, ...):
// degree histogram (integer atomics) and the exponent's partial sum and count of
// each chunk in a fixed order, so the grid does not change any result.  The
// others sum C(d_v, 2) over a chunk of the whole vertex space, the first step of
// the wedge prefix.  Both read row starts only, and a small graph's time is its
// launches: with the wedge sums, the exponent, the clearing and the marking of
// graphs without a wedge in launches of their own, the statistics of 2^18 edges
// took 132 us, together 117 (of which the CSR about 85).  Rows through LDS, coalesced,
// instead of 16 strided reads per thread: this pass over 1.7e7 vertices 255 -> 71 us,
// the wedge prefix 287 -> 42.
__global__ __launch_bounds__(kChunkThreads) void stats_chunks(ChunkArgs a) {
    __shared__ uint32_t s_h[32];
    __shared__ double s_sum[kChunkThreads];
    __shared__ uint64_t s_cnt[kChunkThreads];
    __shared__ uint32_t s_g;
    __shared__ uint64_t s_row[kRowSlots];
    if (blockIdx.x >= a.grid) {
        const uint64_t chunk = blockIdx.x - a.grid;
        load_rows(a.rp, chunk * kChunk, a.nv, s_row);
        __syncthreads();
        uint64_t acc = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int i = (int)threadIdx.x * kPer + j;  // (past the last vertex the rows are equal)
            acc += pairs_of(s_row[row_slot(i + 1)] - s_row[row_slot(i)]);
        }
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
        if ((threadIdx.x & 63) == 0) s_cnt[threadIdx.x >> 6] = acc;
        __syncthreads();
        if (threadIdx.x == 0) a.csum[chunk] = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
        return;
    }
    for (uint64_t c = blockIdx.x; c < a.total; c += a.grid) {
        if (threadIdx.x == 0) s_g = graph_of_chunk(a.G, a.count, c);
        if (threadIdx.x < 32) s_h[threadIdx.x] = 0;
        __syncthreads();
        const StatGraph &g = a.G[s_g];
        const uint64_t v0 = g.v0 + (c - g.chunk0) * kChunk;
        load_rows(a.raw, v0, g.v1, s_row);
        __syncthreads();
        const double denom = (double)g.dmin - 0.5;
        double sum = 0.0;
        uint64_t cnt = 0;
        for (int j = 0; j < kPer; ++j) {
            const int i = (int)threadIdx.x * kPer + j;
            if (v0 + i < g.v1) {
                const uint64_t d = s_row[row_slot(i + 1)] - s_row[row_slot(i)];
                atomicAdd(&s_h[log2_bin(d)], 1u);
                if (d >= g.dmin && d > 0) {
                    sum += log((double)d / denom);
                    ++cnt;
                }
            }
        }
        s_sum[threadIdx.x] = sum;
        s_cnt[threadIdx.x] = cnt;
        __syncthreads();
        for (int off = kChunkThreads / 2; off > 0; off >>= 1) {
            if (threadIdx.x < off) {
                s_sum[threadIdx.x] += s_sum[threadIdx.x + off];
                s_cnt[threadIdx.x] += s_cnt[threadIdx.x + off];
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            a.psum[c] = s_sum[0];
            a.pcnt[c] = s_cnt[0];
        }
        if (threadIdx.x < 32 && s_h[threadIdx.x])
            atomicAdd((unsigned long long *)&a.hist[(uint64_t)g.out * 32 + threadIdx.x],
                      (unsigned long long)s_h[threadIdx.x]);
        __syncthreads();  // s_g, s_h, the rows and the partial sums are reused by the next chunk
    }
}

// Chunk sums to exclusive chunk bases, where there are more than kDirect.
constexpr uint64_t kDirect = 1024;  // chunk sums that every workgroup of the next step adds up itself
__global__ __launch_bounds__(1024) void wedge_chunk_scan(uint64_t *csum, uint64_t nchunks) {
    __shared__ uint64_t s[1024];
    const uint64_t per = (nchunks + 1023) / 1024;
    const uint64_t lo = (uint64_t)threadIdx.x * per, hi = min(lo + per, nchunks);
    uint64_t acc = 0;
    for (uint64_t c = lo; c < hi; ++c) acc += csum[c];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const uint64_t o = threadIdx.x >= (uint32_t)off ? s[threadIdx.x - off] : 0;
        __syncthreads();
        s[threadIdx.x] += o;
        __syncthreads();
    }
    uint64_t run = threadIdx.x > 0 ? s[threadIdx.x - 1] : 0;
    for (uint64_t c = lo; c < hi; ++c) {
        const uint64_t x = csum[c];
        csum[c] = run;
        run += x;
    }
}

// The first `count` workgroups: the exponent of one graph each, from its chunks'
// partials.  The others: the inclusive prefix of C(d_v, 2) over one chunk each.
__global__ __launch_bounds__(kChunkThreads) void stats_apply(ChunkArgs a, double *gamma, bool scanned, uint64_t *pre) {
    __shared__ double s_sum[kChunkThreads];
    __shared__ uint64_t s_cnt[kChunkThreads];
    __shared__ uint64_t s_row[kRowSlots];
    __shared__ uint64_t s_w[2][kChunkThreads / 64];
    const int tid = threadIdx.x;
    if (blockIdx.x < a.count) {
        const StatGraph &g = a.G[blockIdx.x];
        const uint64_t nch = (g.v1 - g.v0 + kChunk - 1) / kChunk;
        double sum = 0.0;
        uint64_t cnt = 0;
        for (uint64_t c = tid; c < nch; c += kChunkThreads) {
            sum += a.psum[g.chunk0 + c];
            cnt += a.pcnt[g.chunk0 + c];
        }
        s_sum[tid] = sum;
        s_cnt[tid] = cnt;
        __syncthreads();
        for (int off = kChunkThreads / 2; off > 0; off >>= 1) {
            if (tid < off) {
                s_sum[tid] += s_sum[tid + off];
                s_cnt[tid] += s_cnt[tid + off];
            }
            __syncthreads();
        }
        if (tid == 0) gamma[g.out] = (s_cnt[0] > 0 && s_sum[0] > 0.0) ? 1.0 + (double)s_cnt[0] / s_sum[0] : (double)NAN;
        return;
    }
    const uint64_t chunk = blockIdx.x - a.count, v0 = chunk * kChunk;
    load_rows(a.rp, v0, a.nv, s_row);
    uint64_t base = 0;
    if (scanned)
        base = tid == 0 ? a.csum[chunk] : 0;
    else
        for (uint64_t c = tid; c < chunk; c += kChunkThreads) base += a.csum[c];
    __syncthreads();
    uint64_t acc = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = tid * kPer + j;
        acc += pairs_of(s_row[row_slot(i + 1)] - s_row[row_slot(i)]);
    }
    uint64_t run = acc;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint64_t y = __shfl_up(run, off, 64);
        if ((tid & 63) >= off) run += y;
    }
    for (int off = 32; off > 0; off >>= 1) base += __shfl_xor(base, off, 64);
    if ((tid & 63) == 63) {
        s_w[0][tid >> 6] = run;
        s_w[1][tid >> 6] = base;
    }
    __syncthreads();
    run -= acc;
#pragma unroll
    for (int w = 0; w < kChunkThreads / 64; ++w) run += (w < (tid >> 6) ? s_w[0][w] : 0) + s_w[1][w];
    // The prefixes take the rows' slots (a thread overwrites the rows that only
    // it still needs: the one after its last is read first) and leave coalesced.
    uint64_t row = s_row[row_slot(tid * kPer)];
    const uint64_t end = s_row[row_slot(tid * kPer + kPer)];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = tid * kPer + j;
        const uint64_t next = j + 1 < kPer ? s_row[row_slot(i + 1)] : end;
        run += pairs_of(next - row);
        row = next;
        s_row[row_slot(i)] = run;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const uint64_t v = v0 + j * kChunkThreads + tid;
        if (v < a.nv) pre[v] = s_row[row_slot(j * kChunkThreads + tid)];
    }
}

// The smallest i in [lo, hi] for which `above` holds (it holds from there on;
// hi: for none below), by LANES consecutive lanes with the same arguments: every
// step asks at LANES places, so it takes log_{LANES + 1} of them.  Whole
// wavefronts call it, a group that need not search with lo = hi.
template <int LANES, typename Above> __device__ __forceinline__ uint64_t first_above(uint64_t lo, uint64_t hi, Above above) {
    const uint32_t lane = threadIdx.x & 63, part = lane % LANES;
    while (LANES == 1 ? lo < hi : __any(lo < hi)) {
        if (LANES == 1) {
            const uint64_t mid = lo + (hi - lo) / 2;
            if (above(mid))
                hi = mid;
            else
                lo = mid + 1;
            continue;
        }
        const uint64_t len = hi - lo, at = lo + len * (part + 1) / (LANES + 1);
        const bool yes = len > 0 && above(at);
        const uint32_t mask = (uint32_t)(__ballot(yes) >> (lane - part)) & ((1u << LANES) - 1);
        const uint32_t first = mask ? (uint32_t)__builtin_ctz(mask) : (uint32_t)LANES;
        const uint64_t up = __shfl(at, (int)(lane - part + (first < LANES ? first : 0)), 64);
        const uint64_t down = __shfl(at, (int)(lane - part + (first > 0 ? first - 1 : 0)), 64);
        if (len > 0) {
            if (first < LANES) hi = up;
            if (first > 0) lo = down + 1;
        }
    }
    return lo;
}

constexpr int kWedgeLanes = 16;  // lanes of a sample, where all of them fit half the GPU at once

struct WedgeArgs {
    const StatGraph *G;
    uint32_t count, samples;
    const uint64_t *rp, *pre;
    const void *col;
    uint32_t key0, key1;
    unsigned long long *closed;  // indexed by StatGraph::out
    uint64_t nv;                 // vertices of the shared space
};

// Sample i of graph g: Philox block (i, 0, 0, WEDGE | gid << 8).  Two searches,
// one load after the other: few samples take LANES lanes each, which shortens
// both (2,000 samples over 16,384 vertices 14.3 us with one lane, 8.3 with 16); from
// the number on whose lanes take half the GPU one lane each is as fast, since the
// samples hide the latency behind one another.  The statistics of 2^18 edges in us
// with one lane / 16: 112.0 / 108.4 for 16,384 samples, 112.0 / 110.3 for 32,768, 112.6 /
// 113.3 for 40,000, 113.8 / 117.1 for 65,536, 116.2 / 123.0 for 100,000.
template <typename IdT, int LANES> __global__ __launch_bounds__(256) void wedge_sample(WedgeArgs a) {
    const uint64_t total_items = (uint64_t)a.count * a.samples;
    const uint64_t stride = (uint64_t)gridDim.x * (256 / LANES);
    const uint64_t it0 = ((uint64_t)blockIdx.x * 256 + threadIdx.x) / LANES, wave0 = it0 - (threadIdx.x & 63) / LANES;
    for (uint64_t step = 0; wave0 + step < total_items; step += stride) {
        const uint64_t it = it0 + step;
        const bool in = it < total_items;
        const StatGraph &g = a.G[in ? it / a.samples : 0];
        const uint32_t i = (uint32_t)(it % a.samples);
        const uint64_t base = g.v0 > 0 ? a.pre[g.v0 - 1] : 0;
        const uint64_t total = g.v1 > g.v0 ? a.pre[g.v1 - 1] - base : 0;
        const bool leader = in && threadIdx.x % LANES == 0;
        if (leader && total == 0 && i == 0) a.closed[g.out] = ~0ull;  // -1: no wedge at all, and no other sample adds to it
        const bool draw = in && total > 0;
        const Block4 w = philox(i, 0, 0, TAG_WEDGE | (g.gid << 8), a.key0, a.key1);
        const uint64_t target = base + uidx64(make_u64(w.w0, w.w1), total);
        // centre: first v with pre[v] > target
        const uint64_t v = first_above<LANES>(g.v0, draw ? g.v1 : g.v0, [&](uint64_t x) { return a.pre[x] > target; });
        const IdT *col = static_cast<const IdT *>(a.col);
        uint64_t lo = 0, hi = 0, nb = 0;
        if (draw) {
            const uint32_t d = (uint32_t)(a.rp[v + 1] - a.rp[v]);
            const uint32_t x = uidx32(w.w2, d);
            uint32_t y = uidx32(w.w3, d - 1);
            if (y >= x) ++y;
            const uint64_t na = (uint64_t)col[a.rp[v] + x];
            nb = (uint64_t)col[a.rp[v] + y];
            // (ids outside the vertex space come only from invalid input; they
            // are never looked up)
            if (na < a.nv) {
                lo = a.rp[na];
                hi = a.rp[na + 1];
            }
        }
        const uint64_t at = first_above<LANES>(lo, hi, [&](uint64_t x) { return (uint64_t)col[x] >= nb; });
        if (leader && at < hi && (uint64_t)col[at] == nb) atomicAdd(&a.closed[g.out], 1ull);
    }
}

__global__ void stats_clear(const StatGraph *G, uint32_t count, uint64_t *hist, long long *closed) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count * 32) return;
    const StatGraph &g = G[i / 32];
    hist[(uint64_t)g.out * 32 + i % 32] = 0;
    if (i % 32 == 0) closed[g.out] = 0;
}

// A single graph's table entry, and its outputs cleared.
__global__ __launch_bounds__(64) void stats_set(StatGraph g, StatGraph *table, uint64_t *hist, long long *closed) {
    const uint32_t i = threadIdx.x;
    if (i < 32) hist[(uint64_t)g.out * 32 + i] = 0;
    if (i == 0) {
        closed[g.out] = 0;
        *table = g;
    }
}

// closed = -1 for a graph with no wedge at all (where no samples are drawn).
__global__ void wedge_mark_empty(const StatGraph *G, uint32_t count, const uint64_t *pre, long long *closed) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const StatGraph &g = G[i];
    const uint64_t base = g.v0 > 0 ? pre[g.v0 - 1] : 0;
    if (g.v1 == g.v0 || pre[g.v1 - 1] == base) closed[g.out] = -1;
}

}  // namespace

uint64_t stats_chunks_of(uint64_t n) { return (n + kChunk - 1) / kChunk; }

size_t stats_scratch_bytes(uint64_t nv, uint64_t total_chunks) {
    const uint64_t vchunks = (nv + kChunk - 1) / kChunk;
    return align256(std::max<uint64_t>(nv, 1) * 8) + align256(std::max<uint64_t>(vchunks, 1) * 8) +
           align256(std::max<uint64_t>(total_chunks, 1) * 8) * 2;
}

int stats_enqueue(StatGraph *G_dev, uint32_t count, uint64_t total_chunks, uint64_t nv, const uint64_t *raw,
                  const uint64_t *rp, const void *col, int id_bytes, uint32_t samples, uint64_t seed, uint64_t *hist,
                  double *gamma, int64_t *closed, void *scratch, hipStream_t s, uint32_t grid, const StatGraph *one) {
    char *p = static_cast<char *>(scratch);
    uint64_t *pre = reinterpret_cast<uint64_t *>(p);
    p += align256(std::max<uint64_t>(nv, 1) * 8);
    const uint64_t vchunks = (nv + kChunk - 1) / kChunk;
    uint64_t *csum = reinterpret_cast<uint64_t *>(p);
    p += align256(std::max<uint64_t>(vchunks, 1) * 8);
    double *psum = reinterpret_cast<double *>(p);
    p += align256(std::max<uint64_t>(total_chunks, 1) * 8);
    uint64_t *pcnt = reinterpret_cast<uint64_t *>(p);
    long long *cl = reinterpret_cast<long long *>(closed);
    if (count == 0) return SFG_OK;
    {
        ProfScope _ps("stats_chunks", s);
        if (one)
            stats_set<<<1, 64, 0, s>>>(*one, G_dev, hist, cl);
        else
            stats_clear<<<(count * 32 + 255) / 256, 256, 0, s>>>(G_dev, count, hist, cl);
    }
    const uint64_t g = std::min<uint64_t>(grid ? grid : total_chunks, total_chunks);
    const ChunkArgs ca{G_dev, count, total_chunks, raw, hist, psum, pcnt, (uint32_t)g, rp, nv, csum};
    if (g + vchunks > 0) {
        ProfScope _ps("stats_chunks", s);
        stats_chunks<<<(unsigned)(g + vchunks), kChunkThreads, 0, s>>>(ca);
    }
    const bool scanned = vchunks > kDirect;
    if (scanned) {
        ProfScope _ps("stats_wedge_scan", s);
        wedge_chunk_scan<<<1, 1024, 0, s>>>(csum, vchunks);
    }
    { ProfScope _ps("stats_gamma", s); stats_apply<<<(unsigned)(count + vchunks), kChunkThreads, 0, s>>>(ca, gamma, scanned, pre); }
    if (samples > 0) {
        WedgeArgs wa{G_dev, count, samples, rp, pre, col, (uint32_t)seed, (uint32_t)(seed >> 32),
                     reinterpret_cast<unsigned long long *>(closed), nv};
        const uint64_t items = (uint64_t)count * samples;
        const uint64_t resident = (uint64_t)device_cu_count() * 16;  // workgroups
        const int lanes = items * kWedgeLanes * 2 <= resident * 256 ? kWedgeLanes : 1;
        const unsigned g = (unsigned)std::max<uint64_t>(1, std::min<uint64_t>((items * lanes + 255) / 256, resident));
        ProfScope _ps("stats_wedge", s);
        if (id_bytes == 4 && lanes > 1)
            wedge_sample<int32_t, kWedgeLanes><<<g, 256, 0, s>>>(wa);
        else if (id_bytes == 4)
            wedge_sample<int32_t, 1><<<g, 256, 0, s>>>(wa);
        else if (lanes > 1)
            wedge_sample<int64_t, kWedgeLanes><<<g, 256, 0, s>>>(wa);
        else
            wedge_sample<int64_t, 1><<<g, 256, 0, s>>>(wa);
    }
    else { ProfScope _ps("stats_wedge", s); wedge_mark_empty<<<(count + 255) / 256, 256, 0, s>>>(G_dev, count, pre, cl); }
    return check_launch("graph statistics");
}

}  // namespace sfg

using namespace sfg;

namespace {
struct GsPlan {
    size_t off_csr, off_rp, off_col, off_table, off_hist, off_scratch, total;
};
GsPlan gs_plan(uint64_t n, uint64_t E, int id_bytes) {
    GsPlan p;
    size_t o = 0;
    auto take = [&](size_t b) {
        size_t r = o;
        o += align256(b);
        return r;
    };
    p.off_csr = take(csr_workspace_bytes(n, E, id_bytes, SFG_CSR_SYMMETRIZE | SFG_CSR_SIMPLE));
    p.off_rp = take((n + 1) * 8);
    p.off_col = take(std::max<uint64_t>(2 * E, 1) * id_bytes);
    p.off_table = take(sizeof(StatGraph));
    p.off_hist = take(0);
    p.off_scratch = take(stats_scratch_bytes(n, stats_chunks_of(n)));
    p.total = o;
    return p;
}
}  // namespace

extern "C" size_t graph_stats_workspace_bytes(uint64_t n, uint64_t num_edges, int id_bytes) {
    if (n == 0 || (id_bytes != 4 && id_bytes != 8)) return 0;
    return gs_plan(n, num_edges, id_bytes).total;
}

extern "C" int graph_stats(uint64_t n, uint64_t num_edges, const void *src, const void *dst, int id_bytes,
                           uint32_t num_samples, uint64_t seed, uint32_t graph_id, uint64_t *degree_hist32,
                           double *gamma, int64_t *closed, void *workspace, size_t workspace_bytes, void *stream) {
    if (n == 0) return fail(SFG_EINVAL, "graph_stats: n must be >= 1");
    if (id_bytes != 4 && id_bytes != 8) return fail(SFG_EINVAL, "graph_stats: id_bytes must be 4 or 8");
    if (!degree_hist32 || !gamma || !closed) return fail(SFG_EINVAL, "graph_stats: NULL output");
    if (num_edges > 0 && (!src || !dst)) return fail(SFG_EINVAL, "graph_stats: NULL edge buffer");
    if (graph_id >= (1u << 24)) return fail(SFG_EINVAL, "graph_stats: graph_id must be < 2^24");
    if (!workspace) return fail(SFG_EINVAL, "graph_stats: workspace is NULL");
    const GsPlan P = gs_plan(n, num_edges, id_bytes);
    if (workspace_bytes < P.total)
        return fail(SFG_ENOSPACE, "graph_stats: workspace has %zu bytes, needs %zu", workspace_bytes, P.total);
    hipStream_t s = as_stream(stream);
    char *ws = static_cast<char *>(workspace);
    uint64_t *rp = reinterpret_cast<uint64_t *>(ws + P.off_rp);
    void *col = ws + P.off_col;
    const uint64_t *raw = nullptr;
    // The CSR's own histogram is the multigraph degree histogram.
    int rc = csr_build(n, num_edges, src, dst, id_bytes, SFG_CSR_SYMMETRIZE | SFG_CSR_SIMPLE, rp, col, degree_hist32,
                       nullptr, ws + P.off_csr, P.off_rp - P.off_csr, s, &raw);
    if (rc != SFG_OK) return rc;
    StatGraph g{0, n, 2 * ((2 * num_edges + n - 1) / n), 0, 0, graph_id};
    StatGraph *tab = reinterpret_cast<StatGraph *>(ws + P.off_table);
    // stats_enqueue recomputes the histogram per graph into degree_hist32.
    return stats_enqueue(tab, 1, stats_chunks_of(n), n, raw, rp, col, id_bytes, num_samples, seed, degree_hist32, gamma,
                         closed, ws + P.off_scratch, s, 0, &g);
}
