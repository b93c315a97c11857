// spkmc_device.hpp -- device-side state, geometry and random numbers of the
// gfx950 spkMC library (host and device code of the library include it; the
// CPU oracle does not).
#pragma once
#include <type_traits>

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "spkmc.h"

#pragma clang fp contract(off)

namespace spkmc {

// Device-resident counters of one lattice, at offset 0 of the caller's buffer.
struct alignas(256) DevState {
    uint64_t cycle;        // cycles completed
    uint64_t fired;        // non-null events
    uint64_t nulls;        // null events
    double t;              // simulated time
    int64_t M;             // sum of spins
    int64_t B;             // sum of nearest-neighbour bond products (each bond once)
    uint64_t rec_count;    // records written (ring index = rec_count % record_cap)
    uint32_t error;        // non-zero: a device-side wait gave up (see kErr*)
    uint32_t pad0;
    uint64_t sums[4];      // per-cycle engine: the one place of its sums over workgroups
    uint64_t pad1[20];
};
static_assert(sizeof(DevState) == 256, "DevState must stay 256 bytes");

enum : uint32_t { kErrBarrierTimeout = 1, kErrFlagTimeout = 2, kErrSelect = 4, kErrHist = 8 };

// Geometry and buffer addresses, passed to every kernel by value.
struct Geom {
    int32_t L, d, h, nd;   // lattice edge, domain edge, octant edge, domains per edge
    int32_t layout;        // SPKMC_LAYOUT_*
    uint32_t K;            // domains
    uint64_t N;            // sites
    uint32_t h2, h3;       // h^2, h^3
    uint32_t wpo;          // PACKED: 32-bit words per octant (h^3 / 32)
    uint32_t fwpo;         // PACKED: halo-copy words per octant (6 h^2 / 32)
    uint32_t rec_cap;
    uint32_t variant;      // SPKMC_VARIANT_* bits
    uint64_t seed;
    DevState *st;
    spkmc_record *rec;
    double *Rk;            // K
    uint32_t *hist;        // 16 words per line: histograms (14 used) of the per-cycle engine; the slots
                           // and flags of the persistent engines; the on-chip launch's exchange words
    uint64_t *flip;        // per-cycle engine: sums over workgroups (cycle_place)
    uint64_t *sync;        // persistent engine: record partials, totals, predictions (PersistScratch)
    uint64_t *dh;          // PACKED: class changes pushed across workgroups, K x 8 octants x 2 spins
    uint32_t *sc;          // PACKED, h = 16: per octant the class counts of its four 4-plane slabs (28 words)
    int8_t *spin8;         // INT8 spins
    uint32_t *A;           // PACKED spins, octant-major, canonical order inside an octant
    uint32_t *F;           // PACKED halo copies: per octant its halo faces x below, x above, y below,
                           // y above, z below, z above (h^2 bits each)
    double r[14];          // rate table
    double rbound;         // R'_max = n_k max_c r_c (RMAX_BOUND)
    uint32_t lpd;          // frequency lines per domain and cycle: 1, or 4 (TWO_COLOURS)
    uint32_t places;       // per-cycle engine: places of its sums (cycle_places)
};

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): two 32x32 -> 64-bit products per round,
// key advanced by the Weyl constants between rounds.
// ---------------------------------------------------------------------------
struct U4 {
    uint32_t x, y, z, w;
};

__host__ __device__ inline U4 philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint64_t key) {
    uint32_t k0 = (uint32_t)key, k1 = (uint32_t)(key >> 32);
#pragma unroll
    for (int i = 0; i < 10; ++i) {
        uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0;
        uint32_t n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return U4{c0, c1, c2, c3};
}

// [0, 1) with 53 random bits
__host__ __device__ inline double unit53(uint32_t a, uint32_t b) {
    return ((double)(a >> 5) * 67108864.0 + (double)(b >> 6)) * (1.0 / 9007199254740992.0);
}
// (0, 1): a 52-bit integer plus one half, over 2^52
__host__ __device__ inline double unit_open52(uint32_t a, uint32_t b) {
    uint64_t m = ((uint64_t)(a >> 6) << 26) | (uint64_t)(b >> 6);
    return ((double)m + 0.5) * (1.0 / 4503599627370496.0);
}
__host__ __device__ inline uint32_t mul_index(uint32_t w, uint32_t n) {
    return (uint32_t)(((uint64_t)w * n) >> 32);
}

// The per-cycle draw shared by every domain: colour (top 3 bits of the first
// word; with two colours its top bit) and the clock uniform.
struct CycleDraw {
    int colour;
    double ut;
};
__host__ __device__ inline CycleDraw cycle_draw(uint64_t seed, uint64_t n, bool two_colours = false) {
    U4 w = philox10((uint32_t)n, (uint32_t)(n >> 32), 0xFFFFFFFFu, 0xFFFFFFFFu, seed);
    return CycleDraw{(int)(w.x >> (two_colours ? 31 : 29)), unit_open52(w.z, w.w)};
}
// Octant of the i-th frequency line (i < 4) of colour c with two colours: the
// octants whose sx + sy + sz has parity c, in increasing order.
__host__ __device__ inline int two_colour_octant(int c, uint32_t i) {
    return c ? (int)((0x7421u >> (4 * i)) & 15u) : (int)((0x6530u >> (4 * i)) & 15u);
}

// Fixed-order FP64 frequency line: separate multiply and add, classes 0..13.
__device__ inline double line_total(const uint32_t *cnt, const double *r) {
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c < 14; ++c) {
        double term = (double)cnt[c] * r[c];
        acc = acc + term;
    }
    return acc;
}
// Class chosen by target = u R_max on the same running sums; -1 = null event.
__device__ inline int line_select(const uint32_t *cnt, const double *r, double target) {
    double acc = 0.0;
    int chosen = -1;
#pragma unroll
    for (int c = 0; c < 14; ++c) {
        double term = (double)cnt[c] * r[c];
        acc = acc + term;
        if (chosen < 0 && target < acc) chosen = c;
    }
    return chosen;
}

__device__ inline double bits_to_double(uint64_t b) { return __longlong_as_double((long long)b); }
__device__ inline uint64_t double_to_bits(double v) { return (uint64_t)__double_as_longlong(v); }

// A value folded over the wavefront, in lane 63 (all lanes take part): DPP shifts within
// each row of 16, then the last lane of each row carried into the rows above; lanes from
// outside read 0.
template <class F>
__device__ inline uint64_t wave_fold(uint64_t v, F f) {
    auto from = [&](auto ctrl, auto rows) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, decltype(ctrl)::value,
                                                                  decltype(rows)::value, 0xF, true);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), decltype(ctrl)::value,
                                                                  decltype(rows)::value, 0xF, true);
        v = f(v, ((uint64_t)hi << 32) | lo);
    };
    using std::integral_constant;
    const integral_constant<int, 0xF> all;
    from(integral_constant<int, 0x111>{}, all);  // row_shr 1, 2, 4, 8
    from(integral_constant<int, 0x112>{}, all);
    from(integral_constant<int, 0x114>{}, all);
    from(integral_constant<int, 0x118>{}, all);
    from(integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});  // row_bcast 15 and 31
    from(integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});
    return v;
}
__device__ inline uint64_t wave_total(uint64_t v) {
    return wave_fold(v, [](uint64_t a, uint64_t b) { return a + b; });
}
__device__ inline uint64_t wave_largest(uint64_t v) {
    return wave_fold(v, [](uint64_t a, uint64_t b) { return a > b ? a : b; });
}

// The per-cycle engine's sums over workgroups (fired, dM, dB, R_max): one place in the
// state header, or, for many workgroups, up to 64 on cache lines of their own in the
// first K words of the flip region, a workgroup adding to place blockIdx mod the count.
// (One place for all took as long as the work at 2048^3: about 20 ns for each of 6144
// atomics per cycle.  But the flip region is a page of its own: 0.5 us for the selection
// and 0.6 for the bookkeeping, more than the atomics of a few workgroups.  256^3 with
// octant edge 8, 16 workgroups: 24.5 us per cycle in the header, 24.9 in 8 places.)  The
// row and slab kernels have 64 to 256 lines to a workgroup: a place for eight of them, from
// 64 on.  The generic ones, which the all-octant maximum may run on, have 1 to 4 (40^3, d = 8,
// two colours, 500 lines: 13 us per cycle in 4 places, 19 in the header).
inline uint32_t cycle_places(const Geom &g) {  // set-up: g.places, and g.flip points to the first
    const bool rows = g.layout == SPKMC_LAYOUT_PACKED && (g.h == 8 || g.h == 16) && !(g.variant & SPKMC_VARIANT_RMAX_ALL);
    const uint32_t per_wg = g.h == 8 ? 256u : g.lpd == 1 ? 64u : 128u;
    const uint32_t lines = g.K * g.lpd, k = rows ? lines / (8 * per_wg) : g.K >> 4;  // at least 16 words a place
    if (rows ? k < 8 : lines < 128 || !k) return 1u;
    return k >= 64 ? 64u : 1u << (31 - __builtin_clz(k));
}
__device__ inline uint64_t *cycle_place(const Geom &g, uint32_t i) { return g.flip + 16 * (i & (g.places - 1)); }
__device__ inline void add_counters(const Geom &g, long long F, long long dM, long long dB) {
    unsigned long long *p = (unsigned long long *)cycle_place(g, blockIdx.x);
    if (F) atomicAdd(&p[0], (unsigned long long)F);
    if (dM) atomicAdd(&p[1], (unsigned long long)dM);
    if (dB) atomicAdd(&p[2], (unsigned long long)dB);
}
__device__ inline void raise_rmax(const Geom &g, unsigned long long bits) {  // R >= 0: ordered as its bits
    atomicMax((unsigned long long *)cycle_place(g, blockIdx.x) + 3, bits);
}
// R_max of the cycle (every lane of the wavefront takes part).
__device__ inline double cycle_rmax(const Geom &g) {
    if (g.variant & SPKMC_VARIANT_RMAX_BOUND) return g.rbound;
    if (g.places == 1) return bits_to_double(g.flip[3]);
    const uint64_t v = wave_largest(cycle_place(g, threadIdx.x & 63)[3]);
    return bits_to_double(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 63) << 32) |
                          (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63));
}

// Step 5 and the bookkeeping of cycle n on the per-cycle engine (one wavefront,
// after every workgroup's selection and flips): the clock, the counters from the
// sums, the observation record; the sums reset.  A launch on every cycle's path: the
// sums and the state travel together.
__device__ inline void finalize_cycle(const Geom &g, uint64_t n, uint32_t obs_every) {
    DevState *st = g.st;
    const bool two = g.lpd == 4;
    const uint32_t places = g.places;
    uint64_t sum[4] = {0, 0, 0, 0};
    uint64_t *const p = cycle_place(g, threadIdx.x);
    if (threadIdx.x < places)
        for (int i = 0; i < 4; ++i) sum[i] = p[i];
    spkmc_record r;
    r.cycle = n + 1;
    r.fired = st->fired;
    r.nulls = st->nulls;
    r.t = st->t;
    r.M = st->M;
    r.B = st->B;
    const CycleDraw cd = cycle_draw(g.seed, n, two);
    const double lnu = -log(cd.ut);
    if (threadIdx.x < places) p[0] = p[1] = p[2] = p[3] = 0;
    if (places > 1) {
        for (int i = 0; i < 3; ++i) sum[i] = wave_total(sum[i]);
        sum[3] = wave_largest(sum[3]);
    }
    if (threadIdx.x != (places > 1 ? 63u : 0u)) return;
    const double Rmax = (g.variant & SPKMC_VARIANT_RMAX_BOUND) ? g.rbound : bits_to_double(sum[3]);
    const uint64_t f = sum[0];
    r.t = r.t + lnu / ((two ? 2.0 : 8.0) * Rmax);
    r.fired += f;
    r.nulls += (uint64_t)g.K * g.lpd - f;
    r.M += (int64_t)sum[1];
    r.B += (int64_t)sum[2];
    st->cycle = r.cycle;
    st->fired = r.fired;
    st->nulls = r.nulls;
    st->t = r.t;
    st->M = r.M;
    st->B = r.B;
    if (obs_every && ((n + 1) % obs_every) == 0 && g.rec_cap) {
        g.rec[st->rec_count % g.rec_cap] = r;
        st->rec_count += 1;
    }
}

// ---------------------------------------------------------------------------
// Site addressing.
// ---------------------------------------------------------------------------
struct OctAddr {
    uint32_t k;
    int s;
    uint32_t q;
};
__device__ inline OctAddr octant_of(const Geom &g, int x, int y, int z) {
    int kx = x / g.d, ky = y / g.d, kz = z / g.d;
    int rx = x - kx * g.d, ry = y - ky * g.d, rz = z - kz * g.d;
    int sx = rx >= g.h, sy = ry >= g.h, sz = rz >= g.h;
    int lx = rx - sx * g.h, ly = ry - sy * g.h, lz = rz - sz * g.h;
    OctAddr a;
    a.k = (uint32_t)kx + (uint32_t)g.nd * ((uint32_t)ky + (uint32_t)g.nd * (uint32_t)kz);
    a.s = sx | (sy << 1) | (sz << 2);
    a.q = (uint32_t)lx + (uint32_t)g.h * ((uint32_t)ly + (uint32_t)g.h * (uint32_t)lz);
    return a;
}

struct Int8Spins {
    __device__ static inline int get(const Geom &g, int x, int y, int z) {
        return g.spin8[(int64_t)x + (int64_t)g.L * ((int64_t)y + (int64_t)g.L * z)];
    }
};
struct PackedSpins {
    __device__ static inline int get(const Geom &g, int x, int y, int z) {
        OctAddr a = octant_of(g, x, y, z);
        uint64_t bit = ((uint64_t)a.k * 8 + (uint64_t)a.s) * g.h3 + a.q;
        return ((g.A[bit >> 5] >> (bit & 31)) & 1u) ? 1 : -1;
    }
};

template <class S>
__device__ inline int aligned_count(const Geom &g, int x, int y, int z, int s) {
    int L = g.L;
    int xm = x ? x - 1 : L - 1, xp = x + 1 == L ? 0 : x + 1;
    int ym = y ? y - 1 : L - 1, yp = y + 1 == L ? 0 : y + 1;
    int zm = z ? z - 1 : L - 1, zp = z + 1 == L ? 0 : z + 1;
    return (S::get(g, xm, y, z) == s) + (S::get(g, xp, y, z) == s) + (S::get(g, x, ym, z) == s) +
           (S::get(g, x, yp, z) == s) + (S::get(g, x, y, zm) == s) + (S::get(g, x, y, zp) == s);
}

// Origin of octant (k, s).
__device__ inline void octant_origin(const Geom &g, uint32_t k, int s, int &ox, int &oy, int &oz) {
    uint32_t nd = (uint32_t)g.nd;
    int kx = (int)(k % nd), ky = (int)((k / nd) % nd), kz = (int)(k / (nd * nd));
    ox = kx * g.d + (s & 1) * g.h;
    oy = ky * g.d + ((s >> 1) & 1) * g.h;
    oz = kz * g.d + ((s >> 2) & 1) * g.h;
}

}  // namespace spkmc
