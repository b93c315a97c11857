// spin_bytes.hpp -- the spins between the caller's bytes and the packed bits of the
// device layout (host code only, plain C++: G is the lattice's geometry, Geom).
#pragma once

#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <thread>
#include <vector>

namespace spkmc {

// ---------------------------------------------------------------------------
// Spins between the caller's bytes (linear order) and the packed bits (octant-
// major), eight sites at a time in linear order, so that the large side, the
// bytes, is read or written once from end to end; layers of octants on a few
// threads where there are many sites (the pages of a new buffer are first touched
// here too).  An octant row is h bits at a multiple of 4 bits (h % 4 == 0).  A
// set, a ten-cycle run and a copy at 240^3 took 129 ms a site at a time, 16 ms so
// on one thread and 3.3 ms on several.
// ---------------------------------------------------------------------------
static const size_t kRowPad = 8;  // bytes past the packed bits that a row's last word may touch
static const uint64_t kOnes = 0x0101010101010101ull;

// Bits of eight +-1 bytes (bit i = byte i is +1); false if a byte is neither.
static inline bool pack8(uint64_t w, uint32_t &bits) {
    const uint64_t neg = (w >> 7) & kOnes;  // 1 where the byte is negative
    bits = (uint32_t)(((neg ^ kOnes) * 0x0102040810204080ull) >> 56);
    return w == (kOnes | neg * 0xFE);
}
static inline uint64_t unpack8(uint32_t bits) {  // the eight bytes of eight bits
    const uint64_t t = ((uint64_t)(bits & 0xFFu) * kOnes) & 0x8040201008040201ull;  // byte i: bit i alone
    const uint64_t up = ((t + 0x7F7F7F7F7F7F7F7Full) >> 7) & kOnes;
    return ~0ull ^ (up * 0xFE);
}
// f(part) for every part < parts (false: a part refused), on up to eight threads, one
// per 2^20 sites.
template <class F>
static bool in_parts(uint64_t parts, uint64_t sites, F f) {
    std::atomic<uint64_t> next{0};
    std::atomic<bool> ok{true};
    auto work = [&]() {
        for (uint64_t i; (i = next.fetch_add(1)) < parts;)
            if (!f(i)) ok = false;
    };
    const uint64_t want = std::min<uint64_t>({8, sites >> 20, std::max(1u, std::thread::hardware_concurrency()), parts});
    std::vector<std::thread> more;
    try {
        more.reserve(8);
        while (more.size() + 1 < want) more.emplace_back(work);
    } catch (...) {  // no more threads to be had: those there are do it all
    }
    work();
    for (std::thread &t : more) t.join();
    return ok;
}
static inline bool valid_spins(const int8_t *s, uint64_t n) {
    const uint64_t chunk = 1u << 20;
    return in_parts((n + chunk - 1) / chunk, n, [=](uint64_t part) {
        const uint64_t end = std::min(n, (part + 1) * chunk);
        uint64_t i = part * chunk, w;
        uint32_t bits;
        bool ok = true;
        for (; i + 8 <= end; i += 8) {
            memcpy(&w, s + i, 8);
            ok &= pack8(w, bits);
        }
        for (; i < end; ++i) ok &= s[i] == 1 || s[i] == -1;
        return ok;
    });
}
// f(first bit of an octant row in the packed order, its first site in linear order)
// for the rows of layer oz of octants
template <class G, class F>
static void for_each_row(const G &g, uint64_t oz, F f) {
    const uint64_t h = (uint64_t)g.h, nd = (uint64_t)g.nd, h3 = g.h3;
    uint64_t site = oz * h * (uint64_t)g.L * (uint64_t)g.L;
    for (uint64_t z = 0; z < h; ++z)
        for (uint64_t oy = 0; oy < 2 * nd; ++oy)
            for (uint64_t y = 0; y < h; ++y) {
                uint64_t bit = (nd * ((oy >> 1) + nd * (oz >> 1)) * 8 + ((oy & 1) << 1 | (oz & 1) << 2)) * h3 + h * (y + h * z);
                for (uint64_t k = 0; k < nd; ++k, bit += 8 * h3, site += 2 * h) {
                    f(bit, site);
                    f(bit + h3, site + h);
                }
            }
}
template <class G>
static bool pack_spins(const G &g, const int8_t *host, unsigned char *A) {
    // A layer's octants are whole bytes that no other layer writes.  A row's last four
    // sites, where it has such, fill the upper half of their byte or the lower: they
    // never reach the next one, which may be another layer's octant on another thread.
    return in_parts(2 * (uint64_t)g.nd, g.N, [=, &g](uint64_t oz) {
        bool ok = true;
        const int h = g.h;
        for_each_row(g, oz, [&](uint64_t bit, uint64_t site) {
            for (int x = 0; x < h; x += 8, bit += 8) {
                uint64_t w = kOnes;  // four sites at the end of a row: the other four count as +1
                uint32_t bits;
                const bool half = h - x < 8;
                memcpy(&w, host + site + x, half ? 4 : 8);
                ok &= pack8(w, bits);
                if (half) bits &= 15u;
                unsigned char *p = A + (bit >> 3);
                bits <<= bit & 7;
                p[0] |= (unsigned char)bits;
                if ((bit & 7) && !half) p[1] |= (unsigned char)(bits >> 8);
            }
        });
        return ok;
    });
}
template <class G>
static void unpack_spins(const G &g, const unsigned char *A, int8_t *host) {
    (void)in_parts(2 * (uint64_t)g.nd, g.N, [=, &g](uint64_t oz) {
        const int h = g.h;
        for_each_row(g, oz, [=](uint64_t bit, uint64_t site) {
            for (int x = 0; x < h; x += 8, bit += 8) {
                const unsigned char *p = A + (bit >> 3);
                const uint64_t w = unpack8((uint32_t)(p[0] | (p[1] << 8)) >> (bit & 7));
                memcpy(host + site + x, &w, h - x < 8 ? 4 : 8);
            }
        });
        return true;
    });
}

}  // namespace spkmc
