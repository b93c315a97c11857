// kernels_resident.hip -- the per-cycle engine's lattices that fit on chip: one
// launch runs many cycles (Sec. 3.1 steps 1-6, Sec. 3.2 steps 4a/4b) with every
// site's state in LDS, for any octant edge, either spin layout and every variant.
//
// What bounds it: a latency chain per cycle (LDS reads, barriers and, with more
// than one workgroup, the R_max exchange); it reads nothing from memory but
// other workgroups' words.  Per cycle, records included: L = 16, d = 8 (one
// workgroup) 2.7 us against 11.4 for three launches per cycle; L = 128, d = 8 (128
// workgroups) 5.7 us against 16.2 (77 while those kernels kept their sums over
// workgroups on one cache line); L = 72, d = 8, two colours 5.2 us against 18.0 (58 then).
//
// Layout in LDS, per domain of the workgroup:
//   * one byte per site, octant-major in canonical order: 8 [up] + (up
//     neighbours).  A flip then changes its own byte by an exclusive or and each
//     neighbour's by +-1, whatever the neighbour's spin, so that flips by
//     different threads commute and every atomic's old value names the class
//     the site left;
//   * per octant the sites of each byte value (16-bit halves of 8 words): the
//     frequency line (step 1) is read from them, nothing is binned.
// A group of GS lanes owns a frequency line: every lane forms the line's sums,
// the group counts the selected byte over its octant's words (GS x W words, a
// contiguous run of W words per lane, W odd so that the lanes fall on different
// LDS banks) and its lanes then move the six neighbours, the site itself, the
// spin in memory and the halo copies, one each.
//
// Between workgroups: the R_max slots of the persistent kernels (bank n & 1,
// generation bit 63), and one 64-bit event record per frequency line (cycle in
// the upper half, bank n & 1).  A workgroup applies the events of the
// neighbouring domains it does not own to its own sites: at the end of the cycle
// where the next colour makes them matter, else while the next maxima travel.
// The records carry their cycle, so no flip has to be waited for.
#include <algorithm>
#include <string>

#include "persistent_common.hpp"
#include "resident.hpp"

namespace spkmc {

namespace {

constexpr uint32_t kPadByte = 15;  // bytes past an octant's last site: a value no class has

struct ResidentHead {
    double r[16];                 // rate of each byte value
    unsigned long long wmax[16];  // per wavefront: its largest line
    unsigned long long stat[4];   // this workgroup's counters of cycle n (bank n & 3)
    double lnu[4];                // -ln u of the clock step of cycle n (place n & 3)
    double rmax;
    int colour[4];                // colour of cycle n (place n & 3)
    int abort;
};
constexpr uint32_t kHeadBytes = 512;
static_assert(sizeof(ResidentHead) <= kHeadBytes, "head");

// class c (7 [up] + aligned) <-> byte value 8 [up] + up neighbours
__device__ __forceinline__ int byte_of_class(int c) { return c >= 7 ? c + 1 : 6 - c; }

constexpr unsigned long long kGenBit = 1ull << 63;

__device__ __forceinline__ uint32_t match_bits(uint32_t w, uint32_t pat) {  // bit 4 of every byte equal to the pattern's
    return (0x10101010u - (w ^ pat)) & 0x10101010u;
}

struct Site {
    int c[3];
};
__device__ __forceinline__ Site site_of(uint32_t q, const ResidentArgs &A) {
    const uint32_t yz = (uint32_t)(((uint64_t)q * A.hinv) >> 32);  // q / h, exact for q < 2^16
    const uint32_t z = (uint32_t)(((uint64_t)yz * A.hinv) >> 32);
    return Site{{(int)(q - yz * (uint32_t)A.g.h), (int)(yz - z * (uint32_t)A.g.h), (int)z}};
}
__device__ __forceinline__ uint32_t index_of(const Site &s, int h) {
    return (uint32_t)(s.c[0] + h * (s.c[1] + h * s.c[2]));
}

// Inclusive prefix sum over the GS lanes of a group.
template <int GS>
__device__ __forceinline__ uint32_t group_scan(uint32_t v) {
    v = row_scan(v);
    if constexpr (GS == 64) {
        v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kRowBcast15, 0xA, 0xF, true);
        v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kRowBcast31, 0xC, 0xF, true);
    }
    return v;
}

// The spin (1 = up) of site (k, o, s) with s possibly one step outside octant o
// along axis `ax`, from the lattice in memory.
__device__ __forceinline__ uint32_t spin_near(const Geom &g, uint32_t k, const int (&kc)[3], int o, Site s, int ax) {
    if (g.layout == SPKMC_LAYOUT_INT8) {
        int X[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            X[a] = kc[a] * g.d + ((o >> a) & 1) * g.h + s.c[a];
            X[a] = X[a] < 0 ? g.L - 1 : X[a] == g.L ? 0 : X[a];
        }
        return g.spin8[(uint32_t)X[0] + (uint32_t)g.L * ((uint32_t)X[1] + (uint32_t)g.L * (uint32_t)X[2])] > 0;
    }
    const int v = ax < 0 ? 0 : s.c[ax];
    if (ax >= 0 && (v < 0 || v == g.h)) {  // the octant's own halo copy
        const int u0 = ax == 0 ? s.c[1] : s.c[0], u1 = ax == 2 ? s.c[1] : s.c[2];
        const uint32_t b = (uint32_t)(2 * ax + (v < 0 ? 0 : 1)) * g.h2 + (uint32_t)(u0 + g.h * u1);
        return (g.F[((uint64_t)k * 8 + (uint64_t)o) * g.fwpo + (b >> 5)] >> (b & 31)) & 1u;
    }
    const uint32_t q = index_of(s, g.h);
    return (g.A[((uint64_t)k * 8 + (uint64_t)o) * g.wpo + (q >> 5)] >> (q & 31)) & 1u;
}

}  // namespace

// GS: lanes per frequency line; MAXT: threads at most (640: the usual 512 of lines and
// two service wavefronts, whose registers do not spill; 1024 spills 46).
template <int GS, int MAXT>
__global__ void __launch_bounds__(MAXT) k_resident(ResidentArgs A) {
    extern __shared__ uint4 lds_raw[];
    const Geom &g = A.g;
    const uint32_t gid = blockIdx.x, G = A.G;
    const uint32_t kbase = gid * A.D;
    const uint32_t nown = kbase >= g.K ? 0u : (g.K - kbase < A.D ? g.K - kbase : A.D);
    const uint32_t lpd = g.lpd, NL = g.K * lpd, lbase = kbase * lpd, nl = nown * lpd;
    const int h = g.h;
    const uint32_t ow = A.ow;
    ResidentHead &sh = *reinterpret_cast<ResidentHead *>(lds_raw);
    uint32_t *const cnt = reinterpret_cast<uint32_t *>(lds_raw) + kHeadBytes / 4;  // [domain][octant][8]
    uint32_t *const nbr = cnt + A.D * 64;                                          // [domain][6]
    uint32_t *const org = nbr + A.D * 6;                                           // [domain]
    uint32_t *const cls = org + A.D;                                               // [domain][octant][ow]
    // one workgroup: the lines' numbers, drawn a cycle ahead [n & 1][line]
    uint4 *const drawn = lds_raw + (kHeadBytes / 4 + A.D * (71 + 8 * ow) + 3) / 4;
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, wave = tid >> 6, nwaves = nthr >> 6;
    const int l = tid & (GS - 1);
    const uint32_t group = (uint32_t)tid / GS, groups = (uint32_t)nthr / GS;
    const bool svc = wave == nwaves - 1;  // records and the clock
    const bool drw = wave == nwaves - 2;  // the draws of the coming cycles
    DevState *const st = g.st;
    const uint64_t n0 = A.n0, n_end = A.n0 + A.ncycles;
    const bool rmax_all = (g.variant & SPKMC_VARIANT_RMAX_ALL) != 0;
    const bool bound = (g.variant & SPKMC_VARIANT_RMAX_BOUND) != 0;
    const double clock_s = lpd == 4 ? 2.0 : 8.0;

    // --- set-up: tables, then every own site's byte from the spins and halos
    if (tid < 16) sh.r[tid] = tid < 7 ? g.r[6 - tid] : tid >= 8 && tid < 15 ? g.r[tid - 1] : 0.0;
    if (tid < 16) sh.wmax[tid] = 0;  // of wavefronts this launch has not
    if (tid == 0) {
        sh.abort = 0;
        sh.stat[0] = sh.stat[1] = sh.stat[2] = sh.stat[3] = 0;
    }
    for (uint32_t i = (uint32_t)tid; i < nown * 6; i += nthr) {
        const int dir = (int)(i % 6), a = dir >> 1;
        const DomainCoord c = dcoord(kbase + i / 6, g.nd);
        int kc[3] = {c.kx, c.ky, c.kz};
        kc[a] = (dir & 1) ? wrapp(kc[a], g.nd) : wrapm(kc[a], g.nd);
        nbr[i] = dindex(kc[0], kc[1], kc[2], g.nd);
    }
    for (uint32_t i = (uint32_t)tid; i < nown; i += nthr) {  // the domain's first site in linear order
        const DomainCoord c = dcoord(kbase + i, g.nd);
        org[i] = (uint32_t)g.d * ((uint32_t)c.kx + (uint32_t)g.L * ((uint32_t)c.ky + (uint32_t)g.L * (uint32_t)c.kz));
    }
    for (uint32_t i = (uint32_t)tid; i < nown * 8 * ow; i += nthr) {
        const uint32_t oct = i / ow, k = kbase + (oct >> 3);
        const int o = (int)(oct & 7u);
        const DomainCoord dc = dcoord(k, g.nd);
        const int kc[3] = {dc.kx, dc.ky, dc.kz};
        uint32_t word = 0;
#pragma unroll 1
        for (int b = 0; b < 4; ++b) {
            const uint32_t q = (i - oct * ow) * 4 + (uint32_t)b;
            uint32_t v = kPadByte;
            if (q < g.h3) {
                const Site s = site_of(q, A);
                v = 8u * spin_near(g, k, kc, o, s, -1);
#pragma unroll
                for (int dir = 0; dir < 6; ++dir) {
                    Site t = s;
                    t.c[dir >> 1] += (dir & 1) ? 1 : -1;
                    v += spin_near(g, k, kc, o, t, dir >> 1);
                }
            }
            word |= v << (8 * b);
        }
        cls[i] = word;
    }
    __syncthreads();
    for (uint32_t ob = 0; ob < nown * 8; ob += groups) {  // every octant's counts, a group each
        const uint32_t oct = ob + group;
        for (int vw = 0; vw < 8; ++vw) {
            uint32_t c0 = 0, c1 = 0;
            if (oct < nown * 8)
                for (uint32_t p = (uint32_t)l; p < ow; p += GS) {
                    const uint32_t w = cls[oct * ow + p];
                    c0 += __builtin_popcount(match_bits(w, 0x02020202u * (uint32_t)vw));
                    if (vw < 7) c1 += __builtin_popcount(match_bits(w, 0x02020202u * (uint32_t)vw + 0x01010101u));
                }
            const uint32_t both = group_scan<GS>(c0 | (c1 << 16));  // a count stays below 2^16
            if (l == GS - 1 && oct < nown * 8) cnt[oct * 8 + vw] = both;
        }
    }

    // a site's byte moves by dn (its neighbour flipped)
    auto bump = [&](uint32_t oct, uint32_t q, int dn) {
        const uint32_t shift = 8 * (q & 3);
        const uint32_t old = (atomicAdd(&cls[oct * ow + (q >> 2)], (uint32_t)dn << shift) >> shift) & 0xFFu;
        const uint32_t now = old + (uint32_t)dn;
        atomicAdd(&cnt[oct * 8 + (old >> 1)], 0u - (1u << (16 * (old & 1))));
        atomicAdd(&cnt[oct * 8 + (now >> 1)], 1u << (16 * (now & 1)));
    };
    // The events of cycle m (colour sp) in neighbouring domains of other workgroups,
    // by threads first, first + step, ...
    auto apply_events = [&](uint64_t m, int sp, uint32_t first, uint32_t step) {
        const uint32_t per = lpd == 1 ? 3u : 12u;
        const uint64_t *bank = A.rec + (m & 1) * (uint64_t)NL;
        for (uint32_t i = first; i < nown * per; i += step) {
            const uint32_t ld = i / per, e = i - ld * per;
            int dir, o;  // the neighbour's direction, and its octant that touches this domain
            if (lpd == 1) {
                dir = 2 * (int)e + (((sp >> e) & 1) ? 0 : 1);
                o = sp;
            } else {
                dir = (int)(e >> 1);
                const int a = dir >> 1, ba = (dir & 1) ? 0 : 1, b1 = (int)(e & 1), b2 = sp ^ ba ^ b1;
                const int x1 = a == 0 ? 1 : 0, x2 = a == 2 ? 1 : 2;
                o = (ba << a) | (b1 << x1) | (b2 << x2);
            }
            const int a = dir >> 1, below = (dir & 1) ? 0 : 1;  // below: the neighbour's upper layer touches
            const uint32_t pk = nbr[ld * 6 + dir];
            if (pk - kbase < nown) continue;
            const uint64_t *p = bank + (lpd == 1 ? pk : 4 * pk + (uint32_t)(o >> 1));
            uint64_t v = ld64(p);
            if ((uint32_t)(v >> 32) != (uint32_t)(m + 1)) {
                const uint64_t start = now_ticks();
                while ((uint32_t)((v = ld64(p)) >> 32) != (uint32_t)(m + 1)) {
                    __builtin_amdgcn_s_sleep(1);
                    if (now_ticks() - start > kTimeoutTicks || ld32(&st->error)) {
                        atomicOr(&st->error, kErrFlagTimeout);
                        sh.abort = 1;
                        break;
                    }
                }
                if ((uint32_t)(v >> 32) != (uint32_t)(m + 1)) break;
            }
            const uint32_t ev = (uint32_t)v;
            if (!(ev >> 31)) continue;
            Site s = site_of(ev & 0xFFFFu, A);
            if (s.c[a] != (below ? h - 1 : 0)) continue;
            s.c[a] = below ? 0 : h - 1;
            bump(ld * 8 + (uint32_t)(o ^ (1 << a)), index_of(s, h), (ev >> 30) & 1u ? -1 : 1);
        }
    };
    // running sums of line f's frequency line (classes in order; with the all-octant
    // maximum the value returned is the largest line among the octants it stands for)
    auto line_oct = [&](uint32_t f, int s) { return lpd == 1 ? s : two_colour_octant(s, f & 3u); };
    auto sums = [&](uint32_t oct, double (&acc)[14]) {
        uint32_t w[8];
        const uint4 *c4 = reinterpret_cast<const uint4 *>(&cnt[oct * 8]);
        const uint4 x = c4[0], y = c4[1];
        w[0] = x.x, w[1] = x.y, w[2] = x.z, w[3] = x.w, w[4] = y.x, w[5] = y.y, w[6] = y.z, w[7] = y.w;
        double a = 0.0;
#pragma unroll
        for (int c = 0; c < 14; ++c) {
            const int v = c >= 7 ? c + 1 : 6 - c;
            const uint32_t cc = (v & 1) ? w[v >> 1] >> 16 : w[v >> 1] & 0xFFFFu;
            const double term = (double)cc * sh.r[v];
            a = a + term;
            acc[c] = a;
        }
        return a;
    };

    // the record keeper's totals since launch start (workgroup 0, service wavefront)
    long long totF = 0, totU = 0, totA = 0;
    const bool keeper = gid == 0 && svc;
    double t = 0.0, t_prev = 0.0;  // the clock now and a cycle ago
    uint64_t fired0 = 0, nulls0 = 0, recs = 0, next_rec = ~0ull;
    int64_t M0 = 0, B0 = 0;
    uint32_t ring = 0;  // the next record's place: recs mod rec_cap
    if (keeper) {
        fired0 = st->fired;
        nulls0 = st->nulls;
        M0 = st->M;
        B0 = st->B;
        t = st->t;
        recs = st->rec_count;
        if (g.rec_cap) ring = (uint32_t)(recs % g.rec_cap);
        if (A.obs_every) next_rec = (n0 / A.obs_every + 1) * A.obs_every;
    }
    // counters of cycle m (packed: fired, of these up spins << 20, sum of aligned counts
    // << 40) into the totals; a whole cycle's fit the fields (fewer than 2^20 lines).
    // Two cycles late, when every workgroup's have arrived: read in the next cycle they
    // kept workgroup 0, and so all, waiting (0.9 us per cycle at L = 128).
    auto gather = [&](uint64_t m) {
        unsigned long long sum = 0;
        if (G == 1) {
            sum = sh.stat[m & 3];
            if (lane == 0) sh.stat[m & 3] = 0;
        } else {
            const unsigned long long gen = ((m >> 2) & 1) << 63;
            const uint64_t *bank = A.part + (m & 3) * (uint64_t)G;
            const uint64_t start = now_ticks();
            for (uint32_t base = 0; base < G; base += 256) {
                unsigned long long v[4];  // in flight together
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t w = base + (uint32_t)(i * 64 + lane);
                    v[i] = w < G ? ld64(&bank[w]) : gen;
                }
                for (;;) {
                    bool all = true;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t w = base + (uint32_t)(i * 64 + lane);
                        if ((v[i] & kGenBit) != gen) {
                            all = false;
                            v[i] = ld64(&bank[w]);
                        }
                    }
                    if (__all(all)) break;
                    __builtin_amdgcn_s_sleep(1);
                    if (now_ticks() - start > kTimeoutTicks || ld32(&st->error)) {
                        atomicOr(&st->error, kErrFlagTimeout);
                        sh.abort = 1;
                        break;
                    }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) sum += v[i] & ~kGenBit;
            }
            for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
        }
        totF += (long long)(sum & 0xFFFFFu);
        totU += (long long)((sum >> 20) & 0xFFFFFu);
        totA += (long long)((sum >> 40) & 0x7FFFFFu);
    };
    // the state after `cyc` cycles: the ring record, or at the end the counters
    auto keep = [&](uint64_t cyc, double at, bool record, bool final) {
        if (lane != 0) return;
        spkmc_record r;
        r.cycle = cyc;
        r.fired = fired0 + (uint64_t)totF;
        r.nulls = nulls0 + (uint64_t)NL * (cyc - n0) - (uint64_t)totF;
        r.t = at;
        r.M = M0 + 2 * totF - 4 * totU;   // an up spin takes 2 from M, a down spin adds 2
        r.B = B0 + 12 * totF - 4 * totA;  // six bonds, `aligned` of them with the old spin
        if (record) {
            g.rec[ring] = r;
            ring = ring + 1 == g.rec_cap ? 0 : ring + 1;
            recs += 1;
        }
        if (final) {
            st->cycle = cyc;
            st->fired = r.fired;
            st->nulls = r.nulls;
            st->t = at;
            st->M = r.M;
            st->B = r.B;
            st->rec_count = recs;
        }
    };

    // the counters of cycle m gathered, and its record appended if one is due (the clock
    // is a cycle ahead)
    auto note = [&](uint64_t m) {
        gather(m);
        if (m + 1 == next_rec) {
            if (g.rec_cap) keep(m + 1, t_prev, true, false);
            next_rec += A.obs_every;
        }
    };
    auto draw = [&](uint64_t n, int colour, uint32_t f) {
        const uint32_t line = lbase + f;
        return philox10((uint32_t)n, (uint32_t)(n >> 32), lpd == 1 ? line : line >> 2, (uint32_t)line_oct(f, colour),
                        g.seed);
    };
    // one workgroup: the numbers of every line for cycle n (with more, each group draws
    // its own while the maxima travel)
    auto draw_lines = [&](uint64_t n, int colour) {
        for (uint32_t f = (uint32_t)lane; f < nl; f += 64) {
            const U4 w = draw(n, colour, f);
            drawn[(n & 1) * nl + f] = uint4{w.x, w.y, w.z, w.w};
        }
    };
    int s = 0, prev = -1;
    if (drw) {
        if (lane < 2) {
            const CycleDraw cd = cycle_draw(g.seed, n0 + (uint64_t)lane, lpd == 4);
            sh.colour[(n0 + (uint64_t)lane) & 3] = s = cd.colour;
            sh.lnu[(n0 + (uint64_t)lane) & 3] = -log(cd.ut);
        }
        if (G == 1) draw_lines(n0, __builtin_amdgcn_readfirstlane(s));
    }
    const bool one = nl <= groups;  // a single round of lines: sums and draws stay in registers
    __syncthreads();
    s = sh.colour[n0 & 3];
    bool pending = false;  // events of the previous cycle (colour prev) still to apply

    for (uint64_t n = n0; n < n_end; ++n) {
        // --- steps 1 and 2: the frequency lines and the workgroup's largest
        double acc[14], m = 0.0;
        for (uint32_t f = group; f < nl; f += groups) {
            const uint32_t dom8 = (lpd == 1 ? f : f >> 2) * 8;
            const int o = line_oct(f, s);
            if (rmax_all)
                for (int oo = 0; oo < 8; ++oo)
                    if (lpd == 1 || oo == (o ^ 1)) m = fmax(m, sums(dom8 + (uint32_t)oo, acc));
            m = fmax(m, sums(dom8 + (uint32_t)o, acc));
        }
        if (!bound) {
            double v = m;
            if constexpr (GS == 16) {  // one value per row
                v = fmax(v, dpp_f64<kRowBcast15, 0xA>(v));
                v = fmax(v, dpp_f64<kRowBcast31, 0xC>(v));
            }
            if (lane == 63) sh.wmax[wave] = double_to_bits(v);
        }
        __syncthreads();
        const uint64_t gen = ((n >> 1) & 1) << 63;
        U4 dw{};
        if (G > 1 && wave == 0) {
            // publish, then poll every workgroup's slot (the fixed bound exchanges zeros:
            // the exchange also keeps the workgroups within a cycle of one another)
            double v = !bound && lane < nwaves ? bits_to_double(sh.wmax[lane < 16 ? lane : 15]) : 0.0;
            v = wave_max_nonneg(v);
            uint64_t *bank = A.slot + A.apart * ((n & 1) * (uint64_t)G);
            if (lane == 63) st64(&bank[A.apart * gid], double_to_bits(v) | gen);
            double best = 0.0;
            const uint64_t start = now_ticks();
            for (uint32_t base = 0; base < G; base += 256) {
                uint64_t sv[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t w = base + (uint32_t)(i * 64 + lane);
                    sv[i] = w < G ? ld64(&bank[A.apart * w]) : gen;
                }
                for (;;) {
                    bool all = true;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t w = base + (uint32_t)(i * 64 + lane);
                        if ((sv[i] & kGenBit) != gen) {
                            all = false;
                            sv[i] = ld64(&bank[A.apart * w]);
                        }
                    }
                    if (__all(all)) break;
                    if (now_ticks() - start > kTimeoutTicks || ld32(&st->error)) {
                        atomicOr(&st->error, kErrBarrierTimeout);
                        sh.abort = 1;
                        break;
                    }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) best = fmax(best, bits_to_double(sv[i] & ~kGenBit));
            }
            best = wave_max_nonneg(best);
            if (lane == 63) sh.rmax = best;
        }
        if (drw) {
            if (G == 1) draw_lines(n + 1, sh.colour[(n + 1) & 3]);
            if (lane == 0) {
                const CycleDraw cd = cycle_draw(g.seed, n + 2, lpd == 4);
                sh.colour[(n + 2) & 3] = cd.colour;
                sh.lnu[(n + 2) & 3] = -log(cd.ut);
            }
        } else if (svc) {
            if (gid == 0 && n > n0 + 1) note(n - 2);
        } else if (wave != 0) {
            if (pending) apply_events(n - 1, prev, (uint32_t)tid - 64, (uint32_t)nthr - 192);
        }
        if (G > 1 && one) dw = draw(n, s, group < nl ? group : 0);
        if (G > 1) {
            __syncthreads();
            if (sh.abort) break;
        }
        double Rmax;
        if (bound) {
            Rmax = g.rbound;
        } else if (G > 1) {
            Rmax = sh.rmax;
        } else {
            double v = bits_to_double(sh.wmax[l & 15]);
            v = fmax(v, dpp_f64<kRowShr1, 0xF>(v));
            v = fmax(v, dpp_f64<kRowShr2, 0xF>(v));
            v = fmax(v, dpp_f64<kRowShr4, 0xF>(v));
            v = fmax(v, dpp_f64<kRowShr8, 0xF>(v));  // lane 15 of each row: the largest of 16
            const uint64_t b = double_to_bits(v);
            Rmax = bits_to_double(((uint64_t)bcast<kRowBcast + 15>((uint32_t)(b >> 32)) << 32) |
                                  bcast<kRowBcast + 15>((uint32_t)b));
        }

        // --- steps 3, 4 and 4b, and the flips
        for (uint32_t fb = 0; fb < nl; fb += groups) {
            const uint32_t f = fb + group;
            const bool valid = f < nl;
            const uint32_t fc = valid ? f : 0;
            const uint32_t ld = lpd == 1 ? fc : fc >> 2;
            const int o = line_oct(fc, s);
            const uint32_t oct = ld * 8 + (uint32_t)o;
            if (G == 1) {
                const uint4 w = drawn[(n & 1) * nl + fc];
                dw = U4{w.x, w.y, w.z, w.w};
            } else if (!one) {
                dw = draw(n, s, fc);
            }
            if (!one) (void)sums(oct, acc);
            const double target = unit53(dw.x, dw.y) * Rmax;
            int cs = -1;
#pragma unroll
            for (int c = 13; c >= 0; --c) cs = target < acc[c] ? c : cs;
            if (!valid) cs = -1;
            // the j-th site of the class in canonical order
            const uint32_t v = (uint32_t)byte_of_class(cs < 0 ? 0 : cs), pat = v * 0x01010101u;
            const uint32_t cw = cnt[oct * 8 + (v >> 1)];
            const uint32_t j = mul_index(dw.z, (v & 1) ? cw >> 16 : cw & 0xFFFFu);
            const uint32_t *const ocls = cls + oct * ow;
            const uint32_t p0 = (uint32_t)l * A.W, p1 = p0 + A.W < ow ? p0 + A.W : ow;
            uint32_t mine = 0;
            for (uint32_t p = p0; p < p1; ++p) mine += __builtin_popcount(match_bits(ocls[p], pat));
            const uint32_t incl = group_scan<GS>(mine), excl = incl - mine;
            const bool here = cs >= 0 && j >= excl && j < incl;
            uint32_t q = 0;
            if (here) {
                uint32_t rank = j - excl;
                uint32_t p = p0, mb = match_bits(ocls[p], pat);
                for (;;) {
                    const uint32_t c = __builtin_popcount(mb);
                    if (rank < c || p + 1 >= p1) break;
                    rank -= c;
                    mb = match_bits(ocls[++p], pat);
                }
                for (; rank; --rank) mb &= mb - 1;
                q = 4 * p + ((uint32_t)__builtin_ctz(mb | 0x80000000u) >> 3);
            }
            uint64_t bal = __ballot(here);
            if constexpr (GS == 16) bal = (bal >> (lane & 48)) & 0xFFFFu;
            const int src = bal ? __builtin_ctzll(bal) : 0;
            q = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(((GS == 16 ? (lane & 48) : 0) + src) << 2), (int)q);
            const bool event = bal != 0;
            if (cs >= 0 && !event && l == 0) atomicOr(&st->error, kErrSelect);  // counts disagree with the bytes
            if (G > 1 && valid && l == 7)
                st64(A.rec + (n & 1) * (uint64_t)NL + lbase + f,
                     ((uint64_t)(uint32_t)(n + 1) << 32) |
                         (event ? 0x80000000u | ((uint32_t)(cs >= 7) << 30) | q : 0u));
            {   // the counters of this wavefront's lines (one lane of each speaks)
                const bool speak = event && l == 0;
                const uint64_t ev = __ballot(speak), ups = __ballot(speak && cs >= 7);
                const uint32_t al = (uint32_t)(cs >= 7 ? cs - 7 : cs);
                unsigned long long sum = (unsigned long long)__popcll(ev) | ((unsigned long long)__popcll(ups) << 20);
#pragma unroll
                for (int b = 0; b < 3; ++b)
                    sum += (unsigned long long)__popcll(__ballot(speak && ((al >> b) & 1u))) << (40 + b);
                if (lane == 0 && sum) atomicAdd(&sh.stat[n & 3], sum);
            }
            if (!event) continue;
            const int up = cs >= 7, dn = up ? -1 : 1;
            const Site sc = site_of(q, A);
            if (l < 7) {
                // the neighbour in direction l, where this workgroup owns it; lane 6: the
                // site itself, whose byte changes by 8
                const int a = l >> 1, side = l & 1;
                Site t = sc;
                uint32_t toct = oct;
                const int x = l == 6 ? 0 : (a == 0 ? sc.c[0] : a == 1 ? sc.c[1] : sc.c[2]) + (side ? 1 : -1);
                int to = x;
                if (l != 6 && (x < 0 || x == h)) {
                    to = side ? 0 : h - 1;
                    uint32_t tl = ld;
                    if (((o >> a) & 1) == side) tl = nbr[ld * 6 + l] - kbase;
                    toct = tl < nown ? tl * 8 + (uint32_t)(o ^ (1 << a)) : ~0u;
                }
                if (a == 0) t.c[0] = to;
                else if (a == 1) t.c[1] = to;
                else if (a == 2) t.c[2] = to;
                if (toct != ~0u) bump(toct, index_of(t, h), l == 6 ? 8 * dn : dn);
            } else if (l == 8) {
                if (g.layout == SPKMC_LAYOUT_INT8) {
                    const uint32_t X = (uint32_t)((o & 1) * h + sc.c[0]), Y = (uint32_t)(((o >> 1) & 1) * h + sc.c[1]);
                    const uint32_t Z = (uint32_t)(((o >> 2) & 1) * h + sc.c[2]);
                    g.spin8[org[ld] + X + (uint32_t)g.L * (Y + (uint32_t)g.L * Z)] = (int8_t)(up ? -1 : 1);
                } else {
                    flip_word(g.A + ((uint64_t)(kbase + ld) * 8 + (uint64_t)o) * g.wpo + (q >> 5), 1u << (q & 31));
                }
            } else if (l >= 9 && l < 12 && g.layout == SPKMC_LAYOUT_PACKED) {
                // the halo copy of the octant across a boundary layer the site lies on
                const int a = l - 9, x = a == 0 ? sc.c[0] : a == 1 ? sc.c[1] : sc.c[2];
                if (x == 0 || x == h - 1) {
                    const int side = x == 0 ? 0 : 1;  // packed octants have h >= 4
                    const uint32_t kt = ((o >> a) & 1) == side ? nbr[ld * 6 + 2 * a + side] : kbase + ld;
                    const int u0 = a == 0 ? sc.c[1] : sc.c[0], u1 = a == 2 ? sc.c[1] : sc.c[2];
                    const uint32_t b = (uint32_t)(2 * a + (side ? 0 : 1)) * g.h2 + (uint32_t)(u0 + h * u1);
                    flip_word(g.F + ((uint64_t)kt * 8 + (uint64_t)(o ^ (1 << a))) * g.fwpo + (b >> 5), 1u << (b & 31));
                }
            }
        }
        // --- step 5, in the record keeper's wavefront (the others need no clock)
        if (svc) {
            t_prev = t;
            t = t + sh.lnu[n & 3] / (clock_s * Rmax);
        }
        // --- step 6: this cycle's events in other workgroups' domains, now where the next
        // cycle's frequency lines can see them (by the wavefronts with no or few lines,
        // while the others flip), else while the next maxima travel
        const int next = sh.colour[(n + 1) & 3], diff = s ^ next;
        pending = G > 1;
        if (G > 1 && n + 1 < n_end && (rmax_all || (lpd == 4 ? diff != 0 : diff && !(diff & (diff - 1))))) {
            pending = false;
            if (wave >= nwaves - 2) apply_events(n, s, (uint32_t)(tid - 64 * (nwaves - 2)), 128u);
        }
        prev = s;
        s = next;
        __syncthreads();
        if (G > 1) {
            if (sh.abort) break;
            if (tid == 0) {
                st64(A.part + (n & 3) * (uint64_t)G + gid, sh.stat[n & 3] | (((n >> 2) & 1) << 63));
                sh.stat[n & 3] = 0;
            }
        }
    }
    __syncthreads();
    if (keeper && !sh.abort) {
        if (A.ncycles > 1) note(n_end - 2);
        gather(n_end - 1);
        if (!sh.abort) keep(n_end, t, n_end == next_rec && g.rec_cap, true);
    }
}

// Slots and counters marked with a generation no cycle of the launch expects first,
// records with a cycle none expects.
__global__ void k_resident_prep(ResidentArgs A) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t NL = (uint64_t)A.g.K * A.g.lpd;
    if (i < 2 * NL) A.rec[i] = A.n0 << 32;
    if (i < A.G)
        for (uint64_t nb = A.n0; nb < A.n0 + 4; ++nb) {
            if (nb < A.n0 + 2) A.slot[A.apart * ((nb & 1) * A.G + i)] = (((nb >> 1) + 1) & 1) << 63;
            A.part[(nb & 3) * A.G + i] = (((nb >> 2) + 1) & 1) << 63;
        }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static void *resident_kernel(int gs, int block) {
    if (block <= 640)
        return gs == 16 ? reinterpret_cast<void *>(&k_resident<16, 640>) : reinterpret_cast<void *>(&k_resident<64, 640>);
    return gs == 16 ? reinterpret_cast<void *>(&k_resident<16, 1024>) : reinterpret_cast<void *>(&k_resident<64, 1024>);
}

bool resident_configure(const Geom &g, ResidentShape &out) {
    out = ResidentShape{};
    // octants of 8 and 16 in packed form have the row and slab kernels; counts are 16-bit
    if (g.layout == SPKMC_LAYOUT_PACKED && (g.h == 8 || g.h == 16)) return false;
    if (g.h3 >= (1u << 16)) return false;
    int dev = 0, cus = 0, lds = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
        return false;
    const uint32_t ow = (g.h3 + 3) / 4;
    const uint64_t per_domain = 64 * 4 + 6 * 4 + 4 + 8ull * ow * 4;
    const uint64_t room = ((uint64_t)lds - kHeadBytes) / per_domain;  // domains one workgroup holds
    if (room == 0) return false;
    const int gs = ow <= 128 ? 16 : 64;
    const uint64_t lines = (uint64_t)g.K * g.lpd;
    if (lines >= (1u << 20)) return false;  // a cycle's packed counters
    // one workgroup while its wavefronts take the lines in two rounds, one with the
    // all-octant maximum (no exchange; launches of one workgroup on several streams run side
    // by side, cooperative ones one after the other: 8 lattices of 32^3, d = 8, on as many
    // threads 10 us per cycle of all so, 38 in two workgroups each, 23 on the per-cycle
    // kernels); else as many as give each a round of kResidentLines lines, up to one per CU.
    // One lattice, us per cycle in one workgroup, in several, and on the per-cycle kernels:
    // 64 lines of 4^3 sites 4.3, 3.9 and 11.4; 125 lines 7.7, 4.0 and 11.6; 256 lines (two
    // colours) 13.7, 4.3 and 12.5; the all-octant maximum 64 lines 8.0, 6.2 and 15.3, 125
    // lines 15.0, 6.3 and 15.6
    const bool all = g.variant & SPKMC_VARIANT_RMAX_ALL;
    uint64_t G = 1;
    if (g.K * per_domain + 32 * lines + 64 > (uint64_t)lds - kHeadBytes || lines * gs > (all ? 1024u : 2048u)) {
        const uint64_t per_wg = gs == 16 ? kResidentLines : 14;  // 14 groups of 64 lanes and the service wavefronts
        G = (lines + per_wg - 1) / per_wg;
        const uint64_t need = (g.K + room - 1) / room;
        G = G < need ? need : G;
        G = G < 2 ? 2 : G;
        G = G > (uint64_t)cus ? (uint64_t)cus : G;
        G = G > g.K ? g.K : G;
    }
    const uint64_t D = (g.K + G - 1) / G;
    if (D > room) return false;
    G = (g.K + D - 1) / D;
    uint64_t thr = D * g.lpd * gs;
    thr = (thr + 63) / 64 * 64 + 128;  // two service wavefronts beside the lines'
    // few lines of large octants: threads for the set-up of every site (about 1.4 us for
    // each site of a thread; a run of two cycles of one domain of 24^3: 96 us with 256
    // threads, 49.5 with 640)
    const uint64_t sites = D * 8 * g.h3;
    const uint64_t least = sites > 32 * 256 ? 640 : 256;
    thr = thr < least ? least : thr > 1024 ? 1024 : thr;
    // Shorter runs take the per-cycle kernels: the set-up against what a cycle saves, in us,
    // fitted to run and observables over 1 to 48 cycles of 53 shapes from 4^3 to 240^3 in
    // four variants.  The set-up: 33 for a cooperative launch, and per site of a thread 1.4
    // (one workgroup of 640 threads) or 1.8, but at least 3 ns per site where the rows of a
    // byte lattice are a power of two apart.  A cycle here takes 2 to 12, in one workgroup
    // 0.04 (0.08) more per line after the first 16; of the per-cycle kernels, 11 and what
    // grows with the lines, and with the longest search for a site among them: over half
    // an octant for one line, and with the fixed bound a line may have no event at all, over
    // a whole one for many.  The maximum over all octants bins eight times as much.  Over
    // those runs no choice is more than 1.12 times slower than the kernels it replaced.
    const bool packed = g.layout == SPKMC_LAYOUT_PACKED, bound = g.variant & SPKMC_VARIANT_RMAX_BOUND;
    const double h3 = (double)g.h3, m = (double)lines, per_thread = (double)sites / (double)thr;
    const double strided = !packed && g.L % (G > 1 ? 64 : 32) == 0 ? 0.003 * (double)sites : 0.0;
    double setup = 7.0 + 1.4 * per_thread + 0.004 * h3;
    if (G > 1 || thr > 640) setup = (G > 1 ? 33.0 : 12.0) + std::max(1.8 * per_thread, strided);
    double saved = (G > 1 ? 7.5 : 8.0) - (bound ? 1.0 : 0.0) + m / 1100.0 + m * h3 * (packed ? 1.5e-5 : 5e-6);
    saved += h3 * (packed ? 0.018 : 0.0075) * m / (m + (bound ? 2.4 : 1.0));
    if (all) saved += 1.5 + h3 * (packed ? 0.0235 : 0.008) + m * h3 * (packed ? 6.5e-5 : 2.1e-5);
    if (G == 1) saved -= (all ? 0.08 : 0.04) * std::max(0.0, m * gs / 16.0 - 16.0);
    if (saved < 0.5) return false;
    out.min_cycles = (uint64_t)(setup / saved) + 1;
    out.G = (int)G;
    out.D = (int)D;
    out.gs = gs;
    out.block = (int)thr;
    out.lds = (size_t)(kHeadBytes + D * per_domain);
    if (G == 1) out.lds += (size_t)(32 * lines + 32);  // the lines' numbers, two cycles of them
    void *kern = resident_kernel(gs, out.block);
    // the limit is the kernel's, for every context that launches it: the device's own
    int occ = 0;
    if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, out.block, out.lds) != hipSuccess || occ < 1) {
        (void)hipGetLastError();
        return false;
    }
    (void)hipGetLastError();
    out.ok = true;
    return true;
}

hipError_t launch_resident(const Geom &g, const ResidentShape &shape, uint64_t n0, uint64_t ncycles,
                           uint32_t obs_every, bool prep, hipStream_t stream) {
    ResidentArgs A;
    A.g = g;
    const uint64_t lines = (uint64_t)g.K * g.lpd;
    // the per-cycle engine's histograms (8 words per line), unused here: two banks of
    // records, then the counters (4 words per workgroup) and the slots (2, each on a cache
    // line of its own where there is room for that, else closer; G <= lines).  Side by side
    // a store took long to arrive through the other workgroups' stores and polls: 7.0 us
    // per cycle at L = 128, d = 8 against 5.7 here.
    A.rec = reinterpret_cast<uint64_t *>(g.hist);
    A.part = A.rec + 2 * lines;
    A.slot = A.part + 4 * (uint64_t)shape.G;
    A.apart = 16;
    while (A.apart > 1 && (4 + 2 * A.apart) * (uint64_t)shape.G > 6 * lines) A.apart /= 2;
    A.n0 = n0;
    A.ncycles = ncycles;
    A.obs_every = obs_every;
    A.G = (uint32_t)shape.G;
    A.D = (uint32_t)shape.D;
    A.ow = (g.h3 + 3) / 4;
    A.W = ((A.ow + (uint32_t)shape.gs - 1) / (uint32_t)shape.gs) | 1u;
    A.hinv = g.h == 1 ? 0u : (uint32_t)(((1ull << 32) + (uint64_t)g.h - 1) / (uint64_t)g.h);
    void *kern = resident_kernel(shape.gs, shape.block);
    void *args[] = {&A};
    if (shape.G == 1)
        return hipLaunchKernel(kern, dim3(1), dim3(shape.block), args, shape.lds, stream);
    if (prep) {
        const uint64_t blocks = (2 * lines + 255) / 256;
        hipLaunchKernelGGL(k_resident_prep, dim3((uint32_t)blocks), dim3(256), 0, stream, A);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipLaunchCooperativeKernel(kern, dim3(shape.G), dim3(shape.block), args, (uint32_t)shape.lds, stream);
}

}  // namespace spkmc
