// kernels_cycle.hip -- state set-up kernels and the per-cycle ("CYCLE" engine)
// kernels of the gfx950 spkMC library.
//
// One cycle (Sec. 3.1 steps 1-6, Sec. 3.2 steps 4a/4b) is three launches:
//   k_bin      one workgroup per frequency line (an active octant): class
//              histogram (step 1), its FP64 frequency line R_k, device-wide
//              max (step 2);
//   k_select   one wavefront per frequency line: draw, frequency-line walk with the
//              null event last (steps 3, 4, 4b), canonical-order prefix select
//              of the site with wavefront ballots, flip (step 6 is the kernel
//              boundary);
//   k_finalize one wavefront: clock (step 5), counters, observation record.
// These kernels are generic over the spin layout and serve as the reference
// launch shape for the persistent engine.
#include <type_traits>

#include "api_internal.hpp"
#include "spkmc_device.hpp"

namespace spkmc {

// --------------------------------------------------------------------------- set-up
__global__ void k_init_int8(Geom g, int init) {
    uint64_t b = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;  // one 128-site block
    uint64_t first = b << 7;
    if (first >= g.N) return;
    U4 w = philox10((uint32_t)b, (uint32_t)(b >> 32), 0xFFFFFFFEu, 0xFFFFFFFEu, g.seed);
    uint32_t words[4] = {w.x, w.y, w.z, w.w};
    for (int i = 0; i < 128 && first + i < g.N; ++i) {
        int v = init == SPKMC_INIT_UP ? 1 : init == SPKMC_INIT_DOWN ? -1 : ((words[i >> 5] >> (i & 31)) & 1u) ? 1 : -1;
        g.spin8[first + i] = (int8_t)v;
    }
}

// The random start of a packed lattice of octant edge H (8 or 16): one thread per
// 128-site block of the linear order, whose Philox words are 128 / H whole octant
// rows, each stored as one H-bit piece (a row starts at a multiple of H, so no
// piece straddles a block).  A thread per packed word instead draws the block of
// each of its rows, every block 128 / H times over: 12.8 ms at 2048^3 against
// 0.97 ms here.
template <int H>
__global__ void k_init_blocks(Geom g) {
    using Piece = std::conditional_t<H == 16, uint16_t, uint8_t>;
    const uint64_t b = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= g.N >> 7) return;
    const U4 w = philox10((uint32_t)b, (uint32_t)(b >> 32), 0xFFFFFFFEu, 0xFFFFFFFEu, g.seed);
    const uint32_t words[4] = {w.x, w.y, w.z, w.w};
    const uint64_t i = b << 7, plane = (uint64_t)g.L * g.L;
    uint32_t z = (uint32_t)(i / plane);
    const uint32_t rem = (uint32_t)(i - z * plane);
    uint32_t y = rem / (uint32_t)g.L, x = rem - y * (uint32_t)g.L;
    Piece *const out = reinterpret_cast<Piece *>(g.A);
#pragma unroll
    for (int p = 0; p < 128 / H; ++p) {
        const uint32_t k = x / (2 * H) + (uint32_t)g.nd * (y / (2 * H) + (uint32_t)g.nd * (z / (2 * H)));
        const uint32_t s = ((x / H) & 1u) | (((y / H) & 1u) << 1) | (((z / H) & 1u) << 2);
        out[((uint64_t)k * 8 + s) * (H * H) + (y % H) + H * (z % H)] =
            (Piece)(words[p * H / 32] >> (p * H % 32));
        x += H;
        if (x == (uint32_t)g.L) {
            x = 0;
            if (++y == (uint32_t)g.L) y = 0, ++z;
        }
    }
}

// One thread per packed word: 32 consecutive canonical sites of one octant.
__global__ void k_init_packed(Geom g, int init) {
    uint64_t wi = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t total = (uint64_t)g.K * 8 * g.wpo;
    if (wi >= total) return;
    uint64_t oct = wi / g.wpo;
    uint32_t k = (uint32_t)(oct >> 3);
    int s = (int)(oct & 7);
    uint32_t q0 = (uint32_t)(wi % g.wpo) * 32;
    int ox, oy, oz;
    octant_origin(g, k, s, ox, oy, oz);
    uint32_t word = 0;
    if (init == SPKMC_INIT_UP) {
        word = 0xFFFFFFFFu;
    } else if (init == SPKMC_INIT_RANDOM) {
        uint64_t cached = ~0ull;
        U4 w{0, 0, 0, 0};
        for (int b = 0; b < 32; ++b) {
            uint32_t q = q0 + b;
            int lx = (int)(q % g.h), ly = (int)((q / g.h) % g.h), lz = (int)(q / g.h2);
            uint64_t i = (uint64_t)(ox + lx) + (uint64_t)g.L * ((uint64_t)(oy + ly) + (uint64_t)g.L * (uint64_t)(oz + lz));
            uint64_t blk = i >> 7;
            if (blk != cached) {
                w = philox10((uint32_t)blk, (uint32_t)(blk >> 32), 0xFFFFFFFEu, 0xFFFFFFFEu, g.seed);
                cached = blk;
            }
            uint32_t src = ((i >> 5) & 3) == 0 ? w.x : ((i >> 5) & 3) == 1 ? w.y : ((i >> 5) & 3) == 2 ? w.z : w.w;
            word |= ((src >> (i & 31)) & 1u) << b;
        }
    }
    g.A[wi] = word;
}

// The octant across face `a` (axis) of octant (k, s): below (side 0) or above
// (side 1), in this domain or the neighbour domain (periodic).
__device__ inline uint64_t octant_across(const Geom &g, uint32_t k, int s, int a, int side) {
    const uint32_t nd = (uint32_t)g.nd;
    uint32_t kc[3] = {k % nd, (k / nd) % nd, k / (nd * nd)};
    const int sa = (s >> a) & 1;
    if (sa == side) kc[a] = side ? (kc[a] + 1 == nd ? 0 : kc[a] + 1) : (kc[a] == 0 ? nd - 1 : kc[a] - 1);
    return ((uint64_t)(kc[0] + nd * (kc[1] + nd * kc[2]))) * 8 + (uint64_t)(s ^ (1 << a));
}

// Halo copies of every octant, rebuilt from the packed spins.  Halo slot f of
// an octant: x below, x above, y below, y above, z below, z above: the layer at
// local coordinate h - 1 of the octant below along the axis (slots 0, 2, 4) or
// layer 0 of the octant above (1, 3, 5).  Inside a slot the bit index is
// (ly + h lz) for x, (lx + h lz) for y, (lx + h ly) for z.
__global__ void k_build_faces(Geom g) {
    uint64_t fw = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t total = (uint64_t)g.K * 8 * g.fwpo;
    if (fw >= total) return;
    uint64_t oct = fw / g.fwpo;
    const uint32_t k = (uint32_t)(oct >> 3);
    const int s = (int)(oct & 7u);
    uint32_t base_bit = (uint32_t)(fw % g.fwpo) * 32;
    uint32_t word = 0;
    for (int b = 0; b < 32; ++b) {
        uint32_t fb = base_bit + b;
        uint32_t f = fb / g.h2, idx = fb % g.h2;
        const int a = (int)(f >> 1), side = (int)(f & 1);
        const uint32_t *srcA = g.A + octant_across(g, k, s, a, side) * g.wpo;
        uint32_t u = idx % g.h, v = idx / g.h, e = side ? 0 : g.h - 1;
        uint32_t lx, ly, lz;
        if (a == 0) { lx = e; ly = u; lz = v; }
        else if (a == 1) { lx = u; ly = e; lz = v; }
        else { lx = u; ly = v; lz = e; }
        uint32_t q = lx + g.h * (ly + g.h * lz);
        word |= ((srcA[q >> 5] >> (q & 31)) & 1u) << b;
    }
    g.F[fw] = word;
}

// The same for octant edges 8 and 16, a word of a face at a time: z faces are words
// of the source octant, y faces its rows (one per plane), x faces one bit of each
// row.  (A bit at a time with run-time divisions: 5.6 ms at 2048^3, this
// 0.66 ms.)
template <int H>
__global__ void k_build_faces_rows(Geom g) {
    constexpr uint32_t FW = H * H / 32, WP = H * H / 32, RW = 32 / H;  // words per face, per plane; rows per word
    const uint64_t fw = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (fw >= (uint64_t)g.K * 8 * 6 * FW) return;
    const uint64_t oct = fw / (6 * FW);
    const uint32_t in = (uint32_t)(fw - oct * (6 * FW)), f = in / FW, j = in % FW;
    const int a = (int)(f >> 1), side = (int)(f & 1);
    const uint32_t *src = g.A + octant_across(g, (uint32_t)(oct >> 3), (int)(oct & 7u), a, side) * (H * WP);
    const uint32_t e = side ? 0u : H - 1;
    uint32_t word = 0;
    if (a == 2) {
        word = src[e * WP + j];
    } else if (a == 1) {
#pragma unroll
        for (uint32_t r = 0; r < RW; ++r)  // row e of planes RW j, RW j + 1, ...
            word |= ((src[(j * RW + r) * WP + e / RW] >> (H * (e % RW))) & ((1u << H) - 1u)) << (H * r);
    } else {
#pragma unroll
        for (uint32_t p = 0; p < H; ++p) {  // rows 32 j .. 32 j + 31 of the octant, RW to a word
            const uint32_t w = src[j * H + p] >> e;
#pragma unroll
            for (uint32_t r = 0; r < RW; ++r) word |= ((w >> (H * r)) & 1u) << (p * RW + r);
        }
    }
    g.F[fw] = word;
}

// M and B of the whole lattice (each bond once: +x, +y, +z of every site): sums
// over the workgroup, then one addition per workgroup.
__device__ void add_observables(const Geom &g, long long m, long long b) {
    __shared__ long long part[2][16];
    for (int o = 32; o > 0; o >>= 1) {
        m += __shfl_xor(m, o);
        b += __shfl_xor(b, o);
    }
    if ((threadIdx.x & 63) == 0) {
        part[0][threadIdx.x >> 6] = m;
        part[1][threadIdx.x >> 6] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (unsigned w = 1; w < blockDim.x >> 6; ++w) {
            m += part[0][w];
            b += part[1][w];
        }
        atomicAdd((unsigned long long *)&g.st->M, (unsigned long long)m);
        atomicAdd((unsigned long long *)&g.st->B, (unsigned long long)b);
    }
}

// INT8: a wavefront per row of sites.
__global__ void k_observables_int8(Geom g) {
    const uint32_t L = (uint32_t)g.L, rows = L * L;
    const uint32_t waves = gridDim.x * (blockDim.x >> 6);
    long long m = 0, b = 0;
    for (uint32_t r = (blockIdx.x * blockDim.x + threadIdx.x) >> 6; r < rows; r += waves) {
        const uint32_t z = r / L, y = r - z * L;
        const int8_t *row = g.spin8 + (uint64_t)r * L;
        const int8_t *ry = g.spin8 + ((uint64_t)z * L + (y + 1 == L ? 0 : y + 1)) * L;
        const int8_t *rz = g.spin8 + ((uint64_t)(z + 1 == L ? 0 : z + 1) * L + y) * L;
        int rm = 0, rb = 0;  // at most L <= 4096 sites
        for (uint32_t x = threadIdx.x & 63; x < L; x += 64) {
            const int v = row[x];
            rm += v;
            rb += v * (row[x + 1 == L ? 0 : x + 1] + ry[x] + rz[x]);
        }
        m += rm;
        b += rb;
    }
    add_observables(g, m, b);
}

// PACKED: M from the set bits, B from the bits that differ from their upper
// neighbour's along each axis (three bonds per site, two less for each that
// differs); the layer above an octant's last one comes from its halo copy.
// Octant edges 8 and 16 a word at a time (a site at a time through the general
// accessor: 62.8 ms at 2048^3 and 127 us at 256^3; this 1.1 ms and 14 us).
template <int H>
__global__ void k_observables_words(Geom g) {
    constexpr uint32_t WP = H * H / 32, WO = H * WP, RW = 32 / H;  // words per plane and octant, rows per word
    constexpr uint32_t kLast = H == 16 ? 0x80008000u : 0x80808080u;  // the last site of every row
    const uint64_t total = (uint64_t)g.K * 8 * WO;
    long long m = 0, b = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t oct = i / WO;
        const uint32_t in = (uint32_t)(i % WO), z = in / WP, p = in % WP;
        const uint32_t *A = g.A + oct * WO;
        const uint32_t *F = g.F + oct * (6 * WP);  // a face holds as many words as a plane
        const uint32_t w = A[in];
        const uint32_t bits = F[WP + (z * H + p * RW) / 32] >> ((z * H + p * RW) % 32);  // x above, rows p RW ...
        uint32_t xh = 0;
#pragma unroll
        for (uint32_t r = 0; r < RW; ++r) xh |= ((bits >> r) & 1u) << (H * r + H - 1);
        const uint32_t wx = ((w >> 1) & ~kLast) | xh;
        // y above: bit lx + H lz of slot 3
        const uint32_t up = p + 1 < WP ? A[in + 1] : F[3 * WP + z / RW] >> (H * (z % RW));
        const uint32_t wy = (w >> H) | (up << (32 - H));
        const uint32_t wz = z + 1 < H ? A[in + WP] : F[5 * WP + p];
        m += 2 * (int)__builtin_popcount(w) - 32;
        b += 96 - 2 * (int)(__builtin_popcount(w ^ wx) + __builtin_popcount(w ^ wy) + __builtin_popcount(w ^ wz));
    }
    add_observables(g, m, b);
}

// Any octant edge: a row of h sites per thread, up to 32 at a time.
__device__ __forceinline__ uint32_t bits_at(const uint32_t *w, uint64_t at, uint32_t n) {  // n <= 32 bits from bit `at`
    const uint32_t sh = (uint32_t)(at & 31);
    uint32_t v = w[at >> 5] >> sh;
    if (sh + n > 32) v |= w[(at >> 5) + 1] << (32 - sh);
    return n == 32 ? v : v & ((1u << n) - 1u);
}
__global__ void k_observables_rows(Geom g) {
    const uint32_t h = (uint32_t)g.h;
    const uint64_t total = (uint64_t)g.K * 8 * g.h2;
    long long m = 0, b = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t oct = i / g.h2;
        const uint32_t in = (uint32_t)(i - oct * g.h2), z = in / h, y = in - z * h;
        const uint32_t *A = g.A + oct * g.wpo, *F = g.F + oct * g.fwpo;
        for (uint32_t x = 0; x < h; x += 32) {
            const uint32_t n = h - x < 32 ? h - x : 32;
            const uint32_t w = bits_at(A, (uint64_t)in * h + x, n);
            const uint32_t next = x + n < h ? bits_at(A, (uint64_t)in * h + x + n, 1) : bits_at(F, g.h2 + in, 1);
            const uint32_t wx = (w >> 1) | (next << (n - 1));
            const uint32_t wy = y + 1 < h ? bits_at(A, (uint64_t)(in + 1) * h + x, n)
                                          : bits_at(F, 3ull * g.h2 + (uint64_t)z * h + x, n);
            const uint32_t wz = z + 1 < h ? bits_at(A, (uint64_t)(in + h) * h + x, n)
                                          : bits_at(F, 5ull * g.h2 + (uint64_t)y * h + x, n);
            m += 2 * (int)__builtin_popcount(w) - (int)n;
            b += 3 * (int)n -
                 2 * (int)(__builtin_popcount(w ^ wx) + __builtin_popcount(w ^ wy) + __builtin_popcount(w ^ wz));
        }
    }
    add_observables(g, m, b);
}

__global__ void k_read_state(const uint64_t *st, uint64_t *host) {
    if (threadIdx.x < sizeof(DevState) / 8) host[threadIdx.x] = st[threadIdx.x];
}

__global__ void k_reset_observables(Geom g) {
    if (threadIdx.x == 0) g.st->M = g.st->B = 0;
}

// The state header, records and scratch before the spins cleared (`words` 64-bit
// words from the start of the buffer), and the rate table written.
__global__ void k_clear(Geom g, uint64_t words) {
    uint64_t *p = reinterpret_cast<uint64_t *>(g.st);
    constexpr uint64_t r0 = sizeof(DevState) / 8;  // the rates follow the header
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = i >= r0 && i < r0 + 14 ? double_to_bits(g.r[i - r0]) : 0ull;
}

// --------------------------------------------------------------------------- cycle
constexpr unsigned kCycleMaxGrid = 1u << 20;  // workgroups of one generic per-cycle launch
// Frequency line f of a cycle: domain f / lpd, octant = the colour (eight
// colours) or the (f mod 4)-th octant of the colour's parity (two colours).
__device__ __forceinline__ void line_of(const Geom &g, uint32_t f, int colour, uint32_t &k, int &s) {
    if (g.lpd == 1) {
        k = f;
        s = colour;
    } else {
        k = f >> 2;
        s = two_colour_octant(colour, f & 3u);
    }
}

template <class S>
__device__ __forceinline__ void bin_octant(const Geom &g, uint32_t k, int s, uint32_t *cnt) {
    int ox, oy, oz;
    octant_origin(g, k, s, ox, oy, oz);
    for (uint32_t q = threadIdx.x; q < g.h3; q += blockDim.x) {
        int x = ox + (int)(q % g.h), y = oy + (int)((q / g.h) % g.h), z = oz + (int)(q / g.h2);
        int sp = S::get(g, x, y, z);
        int c = (sp > 0 ? 7 : 0) + aligned_count<S>(g, x, y, z, sp);
        atomicAdd(&cnt[c], 1u);
    }
}

// Step 1 and the device-wide max of step 2.  One workgroup per frequency line
// (lines f = blockIdx.x, blockIdx.x + gridDim.x, ... when the lines outnumber the
// grid).  RMAX_ALL: the workgroup also bins the inactive octants each line
// stands for (the other seven with eight colours, octant s ^ 1 with two) into
// the maximum; RMAX_BOUND: no maximum is taken.
template <class S>
__global__ void k_bin(Geom g, uint64_t n) {
    __shared__ uint32_t cnt[16];
    const uint32_t lines = g.K * g.lpd;  // < 2^31 (checked at set-up)
    const bool two = g.lpd == 4;
    const CycleDraw cd = cycle_draw(g.seed, n, two);
    double wmax = 0.0;  // thread 0: the largest line of this workgroup
    for (uint32_t f = blockIdx.x; f < lines; f += gridDim.x) {
        uint32_t k;
        int s;
        line_of(g, f, cd.colour, k, s);
        __syncthreads();  // the previous line's counts are read
        if (threadIdx.x < 16) cnt[threadIdx.x] = 0;
        __syncthreads();
        bin_octant<S>(g, k, s, cnt);
        __syncthreads();
        double Rk = 0.0;
        if (threadIdx.x == 0) {
            Rk = line_total(cnt, g.r);
            g.Rk[f] = Rk;
            for (int c = 0; c < 16; ++c) g.hist[(uint64_t)f * 16 + c] = c < 14 ? cnt[c] : 0;
        }
        if (g.variant & SPKMC_VARIANT_RMAX_ALL) {
            for (int o = 0; o < 8; ++o) {
                if (o == s || (two && o != (s ^ 1))) continue;
                __syncthreads();
                if (threadIdx.x < 16) cnt[threadIdx.x] = 0;
                __syncthreads();
                bin_octant<S>(g, k, o, cnt);
                __syncthreads();
                if (threadIdx.x == 0) {
                    double Ro = line_total(cnt, g.r);
                    if (Ro > Rk) Rk = Ro;
                }
            }
        }
        if (Rk > wmax) wmax = Rk;
    }
    if (threadIdx.x == 0 && !(g.variant & SPKMC_VARIANT_RMAX_BOUND) && blockIdx.x < lines)
        raise_rmax(g, double_to_bits(wmax));
}

// Steps 3, 4, 4b and the flip.  One 64-lane wavefront per frequency line, four
// per workgroup (lines f, f + 4 gridDim.x, ... when the lines outnumber the grid).
template <class S>
__global__ void __launch_bounds__(256) k_select(Geom g, uint64_t n) {
    __shared__ long long part[4][3];
    int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint32_t lines = g.K * g.lpd;  // < 2^31 (checked at set-up)
    const CycleDraw cd = cycle_draw(g.seed, n, g.lpd == 4);
    const double Rmax = cycle_rmax(g);
    long long fired = 0, dM = 0, dB = 0;
    for (uint32_t f = blockIdx.x * 4 + wave; f < lines; f += gridDim.x * 4) {
        uint32_t k;
        int so;
        line_of(g, f, cd.colour, k, so);
        U4 dw = philox10((uint32_t)n, (uint32_t)(n >> 32), k, (uint32_t)so, g.seed);
        double target = unit53(dw.x, dw.y) * Rmax;
        uint32_t cnt[14];
        for (int c = 0; c < 14; ++c) cnt[c] = g.hist[(uint64_t)f * 16 + c];
        int cs = line_select(cnt, g.r, target);
        if (cs >= 0) {
            uint32_t j = mul_index(dw.z, cnt[cs]);
            int ox, oy, oz;
            octant_origin(g, k, so, ox, oy, oz);
            for (uint32_t q0 = 0; q0 < g.h3; q0 += 64) {
                uint32_t q = q0 + lane;
                int x = 0, y = 0, z = 0, s = 0, a = 0;
                bool hit = false;
                if (q < g.h3) {
                    x = ox + (int)(q % g.h);
                    y = oy + (int)((q / g.h) % g.h);
                    z = oz + (int)(q / g.h2);
                    s = S::get(g, x, y, z);
                    a = aligned_count<S>(g, x, y, z, s);
                    hit = ((s > 0 ? 7 : 0) + a) == cs;
                }
                uint64_t m = __ballot(hit);
                uint32_t c = (uint32_t)__popcll(m);
                if (j < c) {
                    // lane whose rank among the hits is j
                    uint32_t below = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                    if (hit && below == j) {
                        if (g.layout == SPKMC_LAYOUT_INT8) {
                            g.spin8[(int64_t)x + (int64_t)g.L * ((int64_t)y + (int64_t)g.L * z)] = (int8_t)(-s);
                        } else {
                            uint64_t bit = ((uint64_t)k * 8 + (uint64_t)so) * g.h3 + q;
                            atomicXor(&g.A[bit >> 5], 1u << (bit & 31));
                            // the halo copies of the octants across the boundary layers it lies on
                            const uint32_t c3[3] = {q % g.h, (q / g.h) % g.h, q / g.h2};
                            for (int a = 0; a < 3; ++a) {
                                if (c3[a] != 0 && c3[a] != g.h - 1) continue;
                                for (int side = 0; side < 2; ++side) {
                                    // layer 0 is in the halo above of the octant below (side 0)
                                    if (c3[a] != (side ? g.h - 1 : 0)) continue;
                                    const uint32_t u = a == 0 ? c3[1] : c3[0], v = a == 2 ? c3[1] : c3[2];
                                    const uint32_t b = (uint32_t)(2 * a + (side ? 0 : 1)) * g.h2 + u + g.h * v;
                                    uint32_t *Ft = g.F + octant_across(g, k, so, a, side) * g.fwpo;
                                    atomicXor(&Ft[b >> 5], 1u << (b & 31));
                                }
                            }
                        }
                        fired += 1;
                        dM += -2 * s;
                        dB += 12 - 4 * a;
                    }
                    break;
                }
                j -= c;
            }
        }
    }
    // wavefront sums of the lanes that flipped
    for (int o = 32; o > 0; o >>= 1) {
        fired += __shfl_xor(fired, o);
        dM += __shfl_xor(dM, o);
        dB += __shfl_xor(dB, o);
    }
    if (lane == 0) {
        part[wave][0] = fired;
        part[wave][1] = dM;
        part[wave][2] = dB;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        long long f = 0, m = 0, b = 0;
        for (int w = 0; w < 4; ++w) {
            f += part[w][0];
            m += part[w][1];
            b += part[w][2];
        }
        add_counters(g, f, m, b);
    }
}

// Step 5 and the bookkeeping of cycle n.
__global__ void k_finalize(Geom g, uint64_t n, uint32_t obs_every) {
    finalize_cycle(g, n, obs_every);
}

// --------------------------------------------------------------------------- host launchers
hipError_t launch_clear(const Geom &g, size_t bytes, hipStream_t stream) {
    const uint64_t words = bytes / 8;
    uint64_t blocks = (words + 1023) / 1024;  // four words per thread
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_clear, dim3((unsigned)blocks), dim3(256), 0, stream, g, words);
    return hipGetLastError();
}

hipError_t launch_init(const Geom &g, int init, hipStream_t stream) {
    const uint64_t blocks128 = (g.N + 127) / 128;
    const unsigned grid128 = (unsigned)((blocks128 + 255) / 256);
    if (g.layout == SPKMC_LAYOUT_INT8) {
        hipLaunchKernelGGL(k_init_int8, dim3(grid128), dim3(256), 0, stream, g, init);
    } else if (init == SPKMC_INIT_RANDOM && g.h == 16) {
        hipLaunchKernelGGL(k_init_blocks<16>, dim3(grid128), dim3(256), 0, stream, g);
    } else if (init == SPKMC_INIT_RANDOM && g.h == 8) {
        hipLaunchKernelGGL(k_init_blocks<8>, dim3(grid128), dim3(256), 0, stream, g);
    } else {
        uint64_t words = (uint64_t)g.K * 8 * g.wpo;
        hipLaunchKernelGGL(k_init_packed, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, stream, g, init);
    }
    return hipGetLastError();
}

hipError_t launch_faces(const Geom &g, hipStream_t stream) {
    if (g.layout != SPKMC_LAYOUT_PACKED) return hipSuccess;
    uint64_t fwords = (uint64_t)g.K * 8 * g.fwpo;
    const dim3 grid((unsigned)((fwords + 255) / 256));
    if (g.h == 16) hipLaunchKernelGGL(k_build_faces_rows<16>, grid, dim3(256), 0, stream, g);
    else if (g.h == 8) hipLaunchKernelGGL(k_build_faces_rows<8>, grid, dim3(256), 0, stream, g);
    else hipLaunchKernelGGL(k_build_faces, grid, dim3(256), 0, stream, g);
    return hipGetLastError();
}

hipError_t launch_read_state(const Geom &g, DevState *host, hipStream_t stream) {
    hipLaunchKernelGGL(k_read_state, dim3(1), dim3(64), 0, stream, reinterpret_cast<const uint64_t *>(g.st),
                       reinterpret_cast<uint64_t *>(host));
    return hipGetLastError();
}

hipError_t launch_reset_observables(const Geom &g, hipStream_t stream) {
    hipLaunchKernelGGL(k_reset_observables, dim3(1), dim3(64), 0, stream, g);
    return hipGetLastError();
}

// Adds M and B of the lattice to the state header (zero before).
hipError_t launch_observables(const Geom &g, hipStream_t stream) {
    // items per thread: eight, or more where that many workgroups (each adds to one
    // word of the header) would exceed 1024
    const bool int8 = g.layout == SPKMC_LAYOUT_INT8, words = !int8 && (g.h == 8 || g.h == 16);
    const uint64_t items = int8 ? (uint64_t)g.L * g.L * 64 : words ? g.N / 32 : g.N / (uint64_t)g.h;
    uint64_t blocks = (items + 2047) / 2048;
    if (blocks > 1024) blocks = 1024;
    const dim3 grid((unsigned)blocks);
    if (int8) hipLaunchKernelGGL(k_observables_int8, grid, dim3(256), 0, stream, g);
    else if (g.h == 16) hipLaunchKernelGGL(k_observables_words<16>, grid, dim3(256), 0, stream, g);
    else if (g.h == 8) hipLaunchKernelGGL(k_observables_words<8>, grid, dim3(256), 0, stream, g);
    else hipLaunchKernelGGL(k_observables_rows, grid, dim3(256), 0, stream, g);
    return hipGetLastError();
}

hipError_t launch_cycle(const Geom &g, uint64_t n, uint32_t obs_every, hipStream_t stream, bool slab) {
    if (slab) {
        // PACKED lattices with octant edge 16: the per-cycle slab kernels (their
        // counts binned at the start of the run), then step 5 here
        hipError_t e = launch_cycle_slab(g, n, stream);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_finalize, dim3(1), dim3(64), 0, stream, g, n, obs_every);
        return hipGetLastError();
    }
    if (rows_supported(g)) {
        // PACKED lattices with octant edge 8 or 16: the row kernels, then step 5 here
        hipError_t e = launch_cycle_rows(g, n, stream);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_finalize, dim3(1), dim3(64), 0, stream, g, n, obs_every);
        return hipGetLastError();
    }
    // grids capped well below the 2^32 work-items of one dispatch; the kernels
    // stride over the remaining lines
    const unsigned bin_block = g.h3 >= 256 ? 256 : 64;
    const unsigned lines = g.K * g.lpd;
    const unsigned bin_blocks = lines < kCycleMaxGrid ? lines : kCycleMaxGrid;
    const unsigned sel_blocks = (lines + 3) / 4 < kCycleMaxGrid ? (lines + 3) / 4 : kCycleMaxGrid;
    if (g.layout == SPKMC_LAYOUT_INT8) {
        hipLaunchKernelGGL(k_bin<Int8Spins>, dim3(bin_blocks), dim3(bin_block), 0, stream, g, n);
        hipLaunchKernelGGL(k_select<Int8Spins>, dim3(sel_blocks), dim3(256), 0, stream, g, n);
    } else {
        hipLaunchKernelGGL(k_bin<PackedSpins>, dim3(bin_blocks), dim3(bin_block), 0, stream, g, n);
        hipLaunchKernelGGL(k_select<PackedSpins>, dim3(sel_blocks), dim3(256), 0, stream, g, n);
    }
    hipLaunchKernelGGL(k_finalize, dim3(1), dim3(64), 0, stream, g, n, obs_every);
    return hipGetLastError();
}

}  // namespace spkmc
