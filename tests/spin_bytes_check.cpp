// spin_bytes_check.cpp -- the conversion of spins between bytes and packed bits
// (csrc/spin_bytes.hpp) against one site at a time.
// Usage: spin_bytes_check L d calls; prints the calls that packed or unpacked wrongly.
#include <stdio.h>
#include <stdlib.h>

#include "spin_bytes.hpp"

struct Geom {
    int L, d, h, nd;
    uint64_t N;
    uint32_t h3;
};

// Bit of site (x, y, z): octant-major, domain k, octant s, canonical order inside.
static uint64_t packed_bit(const Geom &g, int x, int y, int z) {
    const int c[3] = {x, y, z};
    uint64_t k = 0, s = 0, q = 0;
    for (int a = 2; a >= 0; --a) {
        const int r = c[a] % g.d;
        k = k * (uint64_t)g.nd + (uint64_t)(c[a] / g.d);
        s |= (uint64_t)(r >= g.h) << a;
        q = q * (uint64_t)g.h + (uint64_t)(r % g.h);
    }
    return (k * 8 + s) * g.h3 + q;
}

int main(int argc, char **argv) {
    if (argc != 4) return 2;
    Geom g{};
    g.L = atoi(argv[1]);
    g.d = atoi(argv[2]);
    g.h = g.d / 2;
    g.nd = g.L / g.d;
    g.N = (uint64_t)g.L * (uint64_t)g.L * (uint64_t)g.L;
    g.h3 = (uint32_t)(g.h * g.h * g.h);
    std::vector<int8_t> spins(g.N), back(g.N);
    const size_t bytes = g.N / 8 + spkmc::kRowPad;
    std::vector<unsigned char> want(bytes, 0), got(bytes);
    uint64_t r = 0x9E3779B97F4A7C15ull, i = 0;
    for (int z = 0; z < g.L; ++z)
        for (int y = 0; y < g.L; ++y)
            for (int x = 0; x < g.L; ++x, ++i) {
                r ^= r << 13, r ^= r >> 7, r ^= r << 17;
                spins[i] = (r >> 40) & 1 ? 1 : -1;
                const uint64_t b = packed_bit(g, x, y, z);
                if (spins[i] > 0) want[b >> 3] |= (unsigned char)(1u << (b & 7));
            }
    int wrong = 0;
    for (int call = 0; call < atoi(argv[3]); ++call) {
        std::fill(got.begin(), got.end(), (unsigned char)0);
        bool ok = spkmc::pack_spins(g, spins.data(), got.data()) && got == want;
        if (call == 0) {
            spkmc::unpack_spins(g, want.data(), back.data());
            ok = ok && back == spins && spkmc::valid_spins(spins.data(), g.N);
            for (const uint64_t at : {(uint64_t)0, g.N / 2 + 3, g.N - 1}) {  // refused wherever it stands
                const int8_t keep = spins[at];
                for (const int8_t bad : {(int8_t)0, (int8_t)2, (int8_t)-2, (int8_t)-128, (int8_t)127}) {
                    spins[at] = bad;
                    std::fill(got.begin(), got.end(), (unsigned char)0);
                    ok = ok && !spkmc::pack_spins(g, spins.data(), got.data()) && !spkmc::valid_spins(spins.data(), g.N);
                }
                spins[at] = keep;
            }
        }
        wrong += !ok;
    }
    printf("%d\n", wrong);
    return 0;
}
