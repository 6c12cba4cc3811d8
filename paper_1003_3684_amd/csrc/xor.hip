// Randomized PK by exclusive OR (PK section, randomization): the adjacency
// matrix of the deterministic Kronecker power XOR that of a random graph.
//
// Only the random graph is sorted: its num_random uniform pair draws are written
// as sort keys, their digits counted as they are drawn, and the CSR build
// merges the sorted pairs with the power's entries, which are in order by
// construction and computed where they are needed (power.hpp).  A pair is kept
// once when exactly one of the two graphs holds it (repeated draws are one
// edge of the random graph).
#include <string.h>

#include <algorithm>

#include "common.hpp"
#include "power.hpp"

namespace sfg {
namespace {

constexpr uint32_t TAG_RANDOM = 6;
constexpr int kXorThreads = 256;
constexpr int kXorCopies = 4;  // interleaved copies of each LDS digit histogram

// Draw i: Philox block (i, 0, 0, tag 6 | gid << 8); row = uidx(w0 + 2^32 w1,
// n), column = uidx(w2 + 2^32 w3, n).
template <typename KeyT>
__global__ __launch_bounds__(kXorThreads) void random_keys(uint64_t count, uint64_t n, uint32_t key0, uint32_t key1,
                                                          uint32_t tagword, int shift, int passes, KeyT *keys,
                                                          uint64_t *hist) {
    __shared__ uint32_t s_h[8 * 256 * kXorCopies];
    for (int i = threadIdx.x; i < passes * 256 * kXorCopies; i += kXorThreads) s_h[i] = 0;
    __syncthreads();
    const uint32_t copy = threadIdx.x % kXorCopies;
    const uint64_t stride = (uint64_t)gridDim.x * kXorThreads;
    for (uint64_t i = (uint64_t)blockIdx.x * kXorThreads + threadIdx.x; i < count; i += stride) {
        const Block4 r = philox((uint32_t)i, (uint32_t)(i >> 32), 0, tagword, key0, key1);
        const KeyT k = ((KeyT)uidx64(make_u64(r.w0, r.w1), n) << shift) | (KeyT)uidx64(make_u64(r.w2, r.w3), n);
        keys[i] = k;
        for (int p = 0; p < passes; ++p) atomicAdd(&s_h[(p * 256 + (uint32_t)((k >> (8 * p)) & 255)) * kXorCopies + copy], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < passes * 256; i += kXorThreads) {
        uint32_t t = 0;
#pragma unroll
        for (int c = 0; c < kXorCopies; ++c) t += s_h[i * kXorCopies + c];
        if (t) atomicAdd((unsigned long long *)&hist[i], (unsigned long long)t);
    }
}

struct XorSizes {
    uint64_t n, e0, epk;
    size_t bytes;
};

int xor_sizes(uint32_t n0, const float *seed_matrix, uint32_t k, uint64_t num_random, int id_bytes, XorSizes *z) {
    if (n0 < 2 || n0 > 64) return fail(SFG_EINVAL, "kron_xor_random: n0 must be in [2, 64]");
    if (k == 0) return fail(SFG_EINVAL, "kron_xor_random: k must be >= 1");
    if (!seed_matrix) return fail(SFG_EINVAL, "kron_xor_random: NULL seed matrix");
    if (id_bytes != 4 && id_bytes != 8) return fail(SFG_EINVAL, "kron_xor_random: id_bytes must be 4 or 8");
    uint64_t e0 = 0;
    for (uint32_t c = 0; c < n0 * n0; ++c) {
        if (!(seed_matrix[c] >= 0.0f) || seed_matrix[c] > 3.0e38f)
            return fail(SFG_EINVAL, "kron_xor_random: bad seed entry %u", c);
        e0 += seed_matrix[c] != 0.0f;
    }
    if (e0 == 0) return fail(SFG_EINVAL, "kron_xor_random: the seed graph has no edge");
    uint64_t n = 1, epk = 1;
    for (uint32_t l = 0; l < k; ++l) {
        if (n > (1ull << 31) / n0) return fail(SFG_ERANGE, "kron_xor_random: n0^k above 2^31");
        n *= n0;
        if (epk > (1ull << 40) / e0) return fail(SFG_ERANGE, "kron_xor_random: e0^k above 2^40");
        epk *= e0;
    }
    if (id_bytes == 4 && n - 1 > 0x7FFFFFFFull) return fail(SFG_ERANGE, "kron_xor_random: ids do not fit int32");
    if (num_random > (1ull << 40)) return fail(SFG_ERANGE, "kron_xor_random: num_random above 2^40");
    // The sort takes one workgroup per tile of entries (see edges_to_csr).
    if (epk + num_random > (1ull << 34)) return fail(SFG_ERANGE, "kron_xor_random: more than 2^34 entries");
    z->n = n;
    z->e0 = e0;
    z->epk = epk;
    z->bytes = csr_xor_workspace_bytes(n, num_random, epk);
    return SFG_OK;
}

}  // namespace
}  // namespace sfg

using namespace sfg;

extern "C" size_t kron_xor_random_workspace_bytes(uint32_t n0, const float *seed_matrix, uint32_t k,
                                                  uint64_t num_random, int id_bytes) {
    XorSizes z;
    return xor_sizes(n0, seed_matrix, k, num_random, id_bytes, &z) == SFG_OK ? z.bytes : 0;
}

extern "C" int kron_xor_random(uint32_t n0, const float *seed_matrix, uint32_t k, uint64_t num_random, uint64_t seed,
                               uint32_t graph_id, int id_bytes, uint64_t *row_ptr, void *col, void *workspace,
                               size_t workspace_bytes, void *stream) {
    XorSizes z;
    int rc = xor_sizes(n0, seed_matrix, k, num_random, id_bytes, &z);
    if (rc != SFG_OK) return rc;
    if (graph_id >= (1u << 24)) return fail(SFG_EINVAL, "kron_xor_random: graph_id must be < 2^24");
    if (!row_ptr || !col) return fail(SFG_EINVAL, "kron_xor_random: NULL output");
    if (!workspace) return fail(SFG_EINVAL, "kron_xor_random: workspace is NULL");
    if (workspace_bytes < z.bytes)
        return fail(SFG_ENOSPACE, "kron_xor_random: workspace has %zu bytes, needs %zu", workspace_bytes, z.bytes);
    hipStream_t s = as_stream(stream);
    Power pw;
    PowerSeed seed_bits;
    make_power(n0, seed_matrix, z.e0, k, pw, seed_bits);
    XorKeys keys;
    rc = csr_xor_begin(z.n, num_random, &pw, seed_bits, row_ptr, workspace, workspace_bytes, s, &keys);
    if (rc != SFG_OK) return rc;
    if (num_random) {
        // (a few workgroups per CU: each adds its counts to the global ones)
        const int g = (int)std::max<uint64_t>(
            1, std::min<uint64_t>((num_random + 16 * kXorThreads - 1) / (16 * kXorThreads), (uint64_t)device_cu_count() * 5));
        const uint32_t key0 = (uint32_t)seed, key1 = (uint32_t)(seed >> 32), tagword = TAG_RANDOM | (graph_id << 8);
        ProfScope _ps("random_pairs", s);
        if (keys.key_bytes == 4)
            random_keys<uint32_t><<<g, kXorThreads, 0, s>>>(num_random, z.n, key0, key1, tagword, keys.shift, keys.passes,
                                                            static_cast<uint32_t *>(keys.keys), keys.hist);
        else
            random_keys<uint64_t><<<g, kXorThreads, 0, s>>>(num_random, z.n, key0, key1, tagword, keys.shift, keys.passes,
                                                            static_cast<uint64_t *>(keys.keys), keys.hist);
    }
    return csr_xor_finish(z.n, num_random, pw, id_bytes, row_ptr, col, workspace, s);
}
