// Prints, for every line "S n nocc trs4" on standard input, the moduli of such
// a purification, the base-2 logarithm of their row limit, and the capacity its
// workspace holds.
#include <cmath>
#include <cstdio>

#include "modular.hpp"

int main() {
    int S, n, nocc, trs4;
    while (std::scanf("%d %d %d %d", &S, &n, &nocc, &trs4) == 4) {
        const int N = dmp::mod_count(S, n, nocc, trs4 != 0);
        std::printf("%d %.17g %d\n", N, N > 0 ? std::log2(dmp::crt_limit(N)) : 0.0, dmp::mod_capacity(S, n));
    }
}
