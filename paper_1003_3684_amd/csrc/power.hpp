// The deterministic Kronecker power of a 0/1 seed (PK section, Kronecker
// product of adjacency matrices) as a sorted sequence of (row, column) pairs
// that is never stored.
//
// Row u of the power has the columns whose digits are, level by level,
// neighbours of u's digits in the seed, so the number of its entries, the
// number of entries in rows below it and the rank of a column among its own are
// products and sums over the levels: the power's entry number g and the number
// of entries at or below a given pair come out of a few steps over small tables.
// Several levels are taken together as one digit of a larger seed (the power of
// the seed by that many levels); the most significant digit takes the levels
// that are left over and has tables of its own.  Two such groupings are used:
// counting looks a pair's digits up in a table of all cells, which is to stay
// small enough for LDS; walking from entry to entry only needs the rows'
// columns, and with larger digits a step is an index and two loads.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

namespace sfg {

constexpr uint32_t kPowerMaxN0 = 64;      // seed vertices
constexpr uint32_t kPowerMaxDigits = 31;  // n0^k <= 2^31
constexpr uint32_t kCountGroup = 32;      // vertices of a digit's seed for counting (a larger seed stays as it is)
constexpr uint32_t kWalkGroup = 1024;     // the same for walking, and
constexpr uint32_t kWalkEntries = 32768;  // its entries

// The digits of one grouping (kernel arguments), digit 0 the most significant.
struct PowerDigits {
    uint32_t digits;
    uint32_t levels[2];                // levels of a digit, [1] of the top one
    uint32_t n[2];                     // vertices of their seeds; n[1] = 0: the top digit is like the others
    uint32_t nmagic;                   // floor((2^32 - 1) / n[0])
    uint32_t place[kPowerMaxDigits];   // vertices below digit l
    uint32_t pmagic[kPowerMaxDigits];  // floor((2^32 - 1) / place)
    uint64_t below[kPowerMaxDigits];   // entries of the digits below l
    uint32_t midplace;                 // place of the digit above the lowest one; 0 if there is none
};

struct PowerSeed {
    uint32_t n0, e0;
    uint32_t mask[kPowerMaxN0 * kPowerMaxN0 / 32];  // nonzero cells, row-major bits
};

// Tables in device memory, built by power_tables ([1]: the top digit's).
struct CountTables {
    uint8_t rank[kPowerMaxN0 * kPowerMaxN0];  // row x, column y: entries of row x below y, + 0x80 if (x, y) is one; the
                                              // second seed's cells follow the first's
    uint16_t start[2][kPowerMaxN0 + 1];       // entries of the rows below x
};
static_assert(2 * kCountGroup * kCountGroup <= kPowerMaxN0 * kPowerMaxN0, "two grouped seeds share the cells");

struct PowerTables {
    CountTables count;
    uint16_t start[2][kWalkGroup + 1];
    uint16_t list[2][kWalkEntries];    // the rows' columns, row after row
    uint16_t rowof[2][kWalkEntries];   // their rows
    uint32_t degmagic[2][kWalkGroup];  // floor((2^32 - 1) / entries of row x)
};

struct Power {
    uint64_t entries;  // e0^k, at most 2^34
    PowerDigits c, w;  // for counting and for walking
    const PowerTables *tables;
};

// Digits of as many levels as keep their seed at max_n vertices and max_e
// entries.
inline void group_levels(uint32_t n0, uint64_t e0, uint32_t k, uint64_t max_n, uint64_t max_e, PowerDigits &p) {
    memset(&p, 0, sizeof(p));
    uint64_t n = n0, e = e0;
    uint32_t g = 1;
    while (g < k && n * n0 <= max_n && e * e0 <= max_e) {
        ++g;
        n *= n0;
        e *= e0;
    }
    const uint32_t top = (k - 1) % g + 1;
    p.digits = (k + g - 1) / g;
    p.levels[0] = g;
    p.levels[1] = top;
    p.n[0] = (uint32_t)n;
    p.n[1] = 0;
    if (top != g)
        for (uint32_t l = p.n[1] = 1; l <= top; ++l) p.n[1] *= n0;
    p.nmagic = 0xFFFFFFFFu / p.n[0];
    p.midplace = p.digits > 1 ? p.n[0] : 0u;
    uint64_t place = 1, below = 1;
    for (uint32_t l = p.digits; l-- > 0;) {
        p.place[l] = (uint32_t)place;
        p.pmagic[l] = (uint32_t)(0xFFFFFFFFu / place);
        p.below[l] = below;
        if (l > 0) {
            place *= n;
            below *= e;
        }
    }
}

// The power of the seed (n0 <= 64 vertices, e0 entries at the nonzero cells)
// by k levels, n0^k <= 2^31, e0^k <= 2^34.
inline void make_power(uint32_t n0, const float *seed, uint64_t e0, uint32_t k, Power &p, PowerSeed &q) {
    memset(&p, 0, sizeof(p));
    memset(&q, 0, sizeof(q));
    q.n0 = n0;
    q.e0 = (uint32_t)e0;
    for (uint32_t c = 0; c < n0 * n0; ++c)
        if (seed[c] != 0.0f) q.mask[c / 32] |= 1u << (c % 32);
    group_levels(n0, e0, k, kCountGroup, ~0ull, p.c);
    group_levels(n0, e0, k, kWalkGroup, kWalkEntries, p.w);
    p.entries = 1;
    for (uint32_t l = 0; l < k; ++l) p.entries *= e0;
}

#if defined(__HIPCC__)

// floor(x / d) by multiply-high with magic = floor((2^32 - 1) / d): the
// estimate is the quotient or one less.
__device__ __forceinline__ uint32_t power_div(uint32_t x, uint32_t d, uint32_t magic) {
    uint32_t q = __umulhi(x, magic);
    if (x - q * d >= d) ++q;
    return q;
}

// Whole workgroup: the counting tables to LDS (the used part).
__device__ __forceinline__ void power_load(const Power &p, CountTables *s) {
    const CountTables &t = p.tables->count;
    const uint32_t cells = p.c.n[0] * p.c.n[0] + p.c.n[1] * p.c.n[1];
    for (uint32_t i = threadIdx.x; i < cells; i += blockDim.x) s->rank[i] = t.rank[i];
    for (uint32_t w = 0; w < 2; ++w)
        for (uint32_t i = threadIdx.x; i <= p.c.n[w]; i += blockDim.x) s->start[w][i] = t.start[w][i];
}

// The number of the power's entries at or below (u, c), both vertices of it;
// *member: whether (u, c) is one.
__device__ __forceinline__ uint64_t power_count(const PowerDigits &p, const CountTables &t, uint32_t u, uint32_t c, bool *member) {
    uint64_t below = 0;     // entries in rows below u
    uint32_t d = 1, r = 0;  // entries that share u's digits so far; columns of u below c so far
    bool in = true;         // c's digits so far are neighbours of u's
    for (uint32_t l = 0; l < p.digits; ++l) {
        const uint32_t w = l == 0 && p.n[1] ? 1u : 0u, n = p.n[w], cell0 = w ? p.n[0] * p.n[0] : 0u;
        const uint32_t place = p.place[l], x = power_div(u, place, p.pmagic[l]), y = power_div(c, place, p.pmagic[l]);
        u -= x * place;
        c -= y * place;
        const uint32_t s = t.start[w][x], deg = t.start[w][x + 1] - s, f = t.rank[cell0 + x * n + y];
        below += (uint64_t)d * s * p.below[l];
        r = r * deg + (in ? f & 0x7Fu : 0u);
        in = in && (f & 0x80u);
        d *= deg;
    }
    *member = in;
    return below + r + (in ? 1u : 0u);
}

// A walk over the power's entries in order.  A row's columns are the sums of
// the columns of its digits, the lowest digit's running fastest: a step moves
// a pointer into that digit's row of the list, and where it wraps one into the
// next digit's.  The column of the entry is rest + *mid p.midplace + *low: the
// two loads are left to the caller, who can issue those of many entries before
// waiting for one.
struct PowerWalk {
    uint32_t u;                              // row
    const uint16_t *low;                     // column of the lowest digit
    uint32_t low_left, low_deg;              // entries of its row from here on, and in all
    const uint16_t *mid;                     // the same for the digit above it (any entry if there is none)
    uint32_t mid_left, mid_deg;
    uint32_t rest;                           // column of the digits above the middle one
    uint32_t i, d;                           // index of `rest` among those of the row, and their number

    // To entry g < entries.
    __device__ __forceinline__ void seek(const PowerDigits &p, const PowerTables &t, uint64_t g) {
        uint32_t rows = 1, x[2] = {0, 0}, s[2] = {0, 0}, deg[2] = {1, 1}, v[2] = {0, 0};  // the last two digits, lowest first
        u = 0;
        for (uint32_t l = 0; l < p.digits; ++l) {
            x[1] = x[0];
            s[1] = s[0];
            deg[1] = deg[0];
            v[1] = v[0];
            v[0] = l == 0 && p.n[1] ? 1u : 0u;
            // Entries below digit l per row of it, times its rows so far: the
            // quotient is an entry of the digit's seed.  (Exact in binary64: g
            // is below 2^34.)
            const uint64_t w = (uint64_t)rows * p.below[l];
            const uint32_t q = (uint32_t)((double)g / (double)w);
            x[0] = t.rowof[v[0]][q];
            s[0] = t.start[v[0]][x[0]];
            deg[0] = t.start[v[0]][x[0] + 1] - s[0];
            g -= w * s[0];
            rows *= deg[0];
            u += x[0] * p.place[l];
        }
        low_deg = deg[0];
        mid_deg = deg[1];
        d = rows / (low_deg * mid_deg);
        uint32_t r = (uint32_t)g;  // index in the row
        uint32_t hi = power_div(r, low_deg, t.degmagic[v[0]][x[0]]);
        const uint32_t il = r - hi * low_deg;
        low = t.list[v[0]] + s[0] + il;
        low_left = low_deg - il;
        mid = t.list[0];
        i = 0;
        rest = 0;
        mid_left = 1;
        if (p.digits == 1) return;
        i = power_div(hi, mid_deg, t.degmagic[v[1]][x[1]]);
        const uint32_t im = hi - i * mid_deg;
        mid = t.list[v[1]] + s[1] + im;
        mid_left = mid_deg - im;
        if (p.digits > 2) above(p, t);
    }
    // rest: the column of index i of row u's digits above the middle one.
    __device__ __forceinline__ void above(const PowerDigits &p, const PowerTables &t) {
        uint32_t uu = power_div(power_div(u, p.n[0], p.nmagic), p.n[0], p.nmagic), ii = i;
        rest = 0;
        for (uint32_t l = p.digits - 2; l-- > 0;) {
            const uint32_t v = l == 0 && p.n[1] ? 1u : 0u;
            const uint32_t uq = l ? power_div(uu, p.n[0], p.nmagic) : 0u, x = uu - uq * p.n[0];
            uu = uq;
            const uint32_t s = t.start[v][x], deg = t.start[v][x + 1] - s;
            const uint32_t iq = l ? power_div(ii, deg, t.degmagic[v][x]) : 0u;
            rest += t.list[v][s + ii - iq * deg] * p.place[l];
            ii = iq;
        }
    }
    // To entry g, the one after the current.
    __device__ __forceinline__ void next(const PowerDigits &p, const PowerTables &t, uint64_t g) {
        ++low;
        if (--low_left) return;
        low -= low_deg;
        low_left = low_deg;
        if (--mid_left) {
            ++mid;
        } else if (++i < d) {
            mid -= mid_deg - 1;
            mid_left = mid_deg;
            above(p, t);
        } else {
            seek(p, t, g);
        }
    }
};

#endif

}  // namespace sfg
