// Host checks of the residue products: the moduli and the Chinese remainder
// constants against 128-bit integers, and the tile lists and the shape rule
// of the planner (modular.hpp, plan.cpp).
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <vector>

#include "plan.hpp"

using namespace dmp;

#define CHECK(x)                                                      \
    do {                                                              \
        if (!(x)) {                                                   \
            std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x);       \
            std::exit(1);                                             \
        }                                                             \
    } while (0)

template <int N>
static void crt() {
    const CrtTable& t = Crt<N>::table;
    __int128 M = 1;
    for (int m = 0; m < N; ++m) {
        for (int q = 0; q < m; ++q) {
            int a = kMods[m], b = kMods[q];
            while (b) std::swap(a %= b, b);
            CHECK(a == 1);
        }
        if (m < 15) M *= kMods[m];   // 15 moduli fit 119 bits
    }
    CHECK(t.limit * t.limit * 2.0 < (t.mh + t.ml) * 0x1p80);
    if (N > 15) return;
    std::mt19937_64 rng(N);
    for (int i = 0; i < 2000; ++i) {
        // integers of every size up to M / 2, both signs
        __int128 x = (__int128(rng() >> 1) << 62) ^ __int128(rng());
        x %= M / 2;
        x >>= rng() % 100;
        if (i == 0) x = M / 2 - M / 8192;
        if (i & 1) x = -x;
        double f0 = -t.k0, f1 = -t.k1;
        for (int m = 0; m < N; ++m) {
            int r = int(x % kMods[m]);
            if (r > kMods[m] / 2 || (kMods[m] == 256 && r == 128)) r -= kMods[m];
            if (r < -(kMods[m] / 2)) r += kMods[m];
            CHECK(r >= -128 && r <= 127);
            f0 = std::fma(double(r + 128), t.w0[m], f0);
            f1 = std::fma(double(r + 128), t.w1[m], f1);
        }
        const double k = std::rint(std::fma(f1, 0x1p-80, f0 * 0x1p-40));
        const double y = std::fma(std::fma(k, -0x1p40, f0), 0x1p40, f1);
        const double got = std::fma(y, t.mh, y * t.ml);
        // the fraction is off by less than 2^-69 (M of it), the rest by a few
        // roundings
        const double want = double(x);
        CHECK(std::fabs(got - want) <= std::ldexp(t.mh, 80 - 69) + 4 * 0x1p-53 * std::fabs(want));
    }
}

int main() {
    crt<11>();
    crt<12>();
    crt<13>();
    crt<14>();
    crt<15>();
    crt<16>();
    for (int S = 1; S <= 12; ++S) {
        CHECK((mod_capacity(S) > 0) == (S >= 6 && S <= 8));
        for (int n : {1, 7, 100, 1000, 20000})
            for (int occ : {0, 1, n / 250, n / 7, n / 2, n})
                CHECK(mod_count(S, n, occ) <= mod_capacity(S) && (mod_capacity(S) == 0 || mod_count(S, n, occ) >= kModMin));
    }
    // every 32 x 32 block on or above the diagonal (all blocks of a full
    // product) lies in exactly one tile of every modulus
    for (int n : {1, 31, 64, 127, 128, 129, 255, 257, 700, 1030})
        for (int shape : {kShapeWide, kShapeSmall})
            for (bool upper : {false, true}) {
                std::vector<Tile> tiles;
                append_residue_tiles(tiles, n, 3, shape, upper, 5);
                CHECK(int(tiles.size()) == 3 * residue_tile_count(n, shape, upper));
                std::set<std::pair<uint32_t, std::pair<int, int>>> seen;
                for (const Tile& t : tiles) {
                    CHECK((t.mat & 0xffffffu) == 5 && (t.mat >> 24) < 3);
                    CHECK(seen.insert({t.mat >> 24, {t.I, t.J}}).second);
                    CHECK(t.I * shape_edge(shape) < n && t.J * shape_edge(shape) < n);
                    CHECK(!upper || t.I <= t.J);
                }
            }
    // few or mostly empty wide tiles: the small shape
    auto shape = [](std::vector<int> n) { return residue_shape(int(n.size()), n.data(), 13, true); };
    CHECK(shape({64}) == kShapeSmall && shape({700}) == kShapeSmall);
    CHECK(shape({1024}) == kShapeWide && shape({2048}) == kShapeWide && shape({8192}) == kShapeWide);
    CHECK(shape(std::vector<int>(40, 100)) == kShapeSmall);
    CHECK(shape(std::vector<int>(24, 1000)) == kShapeWide);
    std::printf("residue plan ok\n");
}
