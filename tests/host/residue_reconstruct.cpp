// The reconstruction from 16 residues against 128-bit integers (their product is
// below 2^126), and the byte a residue comes from for operands beyond the 53 bits of
// FP64's integers.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "modular.hpp"

using namespace dmp;

#define CHECK(x)                                                \
    do {                                                        \
        if (!(x)) {                                             \
            std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x); \
            std::exit(1);                                       \
        }                                                       \
    } while (0)

int main() {
    constexpr int N = 16;
    const CrtTable& t = Crt<N>::table;
    __int128 M = 1;
    for (int m = 0; m < N; ++m) M *= kMods[m];
    CHECK(M > 0);
    const double md = std::ldexp(t.mh, 80);
    // M in two doubles: the remainder, below 2^73, to its own 53 bits
    const __int128 off = __int128(md) + __int128(std::ldexp(t.ml, 80)) - M;
    CHECK(off <= (1 << 20) && -off <= (1 << 20));
    std::mt19937_64 rng(16);
    for (int i = 0; i < 20000; ++i) {
        __int128 x = (__int128(rng() >> 2) << 64) ^ __int128(rng());
        x %= M / 2;
        x >>= rng() % 110;
        if (i == 0) x = M / 2 - M / 8192;
        if (i & 1) x = -x;
        double f0 = -t.k0, f1 = -t.k1;
        for (int m = 0; m < N; ++m) {
            int r = int(x % kMods[m]);
            if (r < 0) r += kMods[m];
            if (r > 127) r -= kMods[m];
            f0 = std::fma(double(r + 128), t.w0[m], f0);
            f1 = std::fma(double(r + 128), t.w1[m], f1);
        }
        const double k = std::rint(std::fma(f1, 0x1p-80, f0 * 0x1p-40));
        const double y = std::fma(std::fma(k, -0x1p40, f0), 0x1p40, f1);
        const double got = std::fma(y, t.mh, y * t.ml);
        // the fraction is off by less than 255 N 2^-81 < 2^-69, the rest by a few roundings
        CHECK(std::fabs(got - double(x)) <= std::ldexp(t.mh, 80 - 69) + 4 * 0x1p-53 * std::fabs(double(x)));
    }
    // the byte of a residue (store_residues): z = xh (2^27 mod p) + xl, q the nearest
    // integer of z / p, for integers up to the row limit of 16 moduli
    for (int i = 0; i < 200000; ++i) {
        double x = std::rint(std::ldexp(double(rng() >> 11), int(rng() % 10)));   // 53 bits, up to 2^62
        if (x > t.limit) x = std::rint(t.limit);
        if (i & 1) x = -x;
        const double xh = std::rint(x * 0x1p-27), xl = std::fma(xh, -0x1p27, x);
        for (int m = 0; m < N; ++m) {
            const int p = kMods[m], c0 = (1 << 27) % p, c = c0 > p / 2 ? c0 - p : c0;
            const double z = std::fma(xh, double(c), xl);
            CHECK(std::fabs(z) < 0x1p43);
            const double magic = 0x1.8p52, inv = 1.0 / p;
            const double q = std::fma(z, inv, magic) - magic, r = z - q * p;
            const __int128 want = __int128(x) % p;
            CHECK(std::fabs(r) <= p / 2);
            CHECK((__int128(r) - want) % p == 0);
        }
    }
    std::printf("reconstruction ok\n");
}
