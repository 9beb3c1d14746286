// Products through residues (the multi-modulus form of the error-free
// scheme): the operands of C = A B become integers X_i = rint(a_i 2^(s_i)),
// one power of two per row of A and per column of B, small enough that
// 2 |(X Y)_ij| < M = p_1 ... p_N for pairwise coprime p_m <= 256; the N
// residue products X Y mod p_m are INT8 (or FP16) matrix products with exact
// sums, and the Chinese remainder theorem gives the integer (X Y)_ij back.
// Nothing is dropped: the only errors are the rounding to X, Y and the final
// rounding to FP64.  Against S digit slices with S (S + 1) / 2 products per
// element this takes N products; kModCount states N.
//
// Shared by host and device code (no HIP calls).
#pragma once

#include <cstdint>

namespace dmp {

constexpr int kMaxMods = 16;
// The largest pairwise coprime integers up to 256, so that balanced residues
// fit a signed byte.
constexpr int kMods[kMaxMods] = {256, 255, 253, 251, 247, 241, 239, 233,
                                 229, 227, 223, 217, 211, 199, 197, 193};

// Slice counts whose purification products run through residues, and the
// moduli of each at large n: 11, 13 and 15 products against 21, 28 and 36.
// S <= 5 and S >= 9 keep the digit slices: below 6 the slices are few enough (15
// products) and their truncation is what is studied; beyond 8 the integers no
// longer fit FP64.
constexpr int kModSlicesLo = 6, kModSlicesHi = 8;
constexpr int kModCount[3] = {11, 13, 15};
constexpr int kModMin = 11;

// Moduli of a purification with S slices, nocc of n levels occupied: the
// smallest count whose error is no larger than that of S digit slices.  Those
// keep 8S - 2 bits of a row below its largest entry m_i, but drop the slice
// pairs i + j > S + 1, which leaves about 2^(8 - 8S) m_i m_j sqrt(n); the
// rounding to X, Y leaves |row i| |row j| / sqrt(M).  In a density matrix of
// filling f the maxima are about f and the row norms sqrt(f), so the quotient of
// the two errors goes as 1 / (f sqrt(n)) = sqrt(n) / nocc.  Measured as whole
// purifications against 11 slices (Frobenius norm of the difference, medians
// over seeds; Haar-distributed and nearly diagonal projectors, n = 8 .. 2048, f =
// 0.03 .. 0.9), residues over slices: canonical, 13 moduli, S = 7, at most 4.5
// sqrt(n) / nocc (f = 0.2, where the slices' powers of two lie closest to the
// maxima), e.g. 2.3 at n = 64, f = 0.2; 1.2 at n = 300, f = 0.2; 0.24 at n =
// 2048, f = 0.25; TRS4 5.6 sqrt(n) / nocc; each modulus more takes it down by 14
// (n = 64, f = 0.2: 0.19).  From half filling on, the maxima pass 1/2 and the
// slices' powers of two double: 0.60 at n = 64, f = 0.5.  S = 6 and 11 moduli:
// the same quotients less a seventh.  The lines below stand a quarter of the
// error above 1: nocc^2 >= 32 n (TRS4 50 n), or half filling and n >= 64 (TRS4
// 100).  Fillings below 15 % and 0.4 % take one and two moduli more at any n.
// S = 8: FP64 rounding is the larger error with 15 moduli as with 16 and with
// slices (against refined eigenvectors, n = 16 .. 64, quotients 0.93 .. 1.12).
constexpr int mod_count(int S, int n, int nocc, bool trs4 = false) {
    if (S < kModSlicesLo || S > kModSlicesHi) return 0;
    const int64_t occ = nocc, levels = n;
    int more = (occ * 100 < levels * 15 ? 1 : 0) + (occ * 1000 < levels * 4 ? 1 : 0);
    const bool half = 2 * occ + 1 >= levels && n >= (trs4 ? 100 : 64);
    if (S < 8 && !half) {
        // one modulus: 14^2 in the square
        int64_t lhs = (occ > 0 ? occ * occ : 1), rhs = (trs4 ? 50 : 32) * levels;
        int steps = 0;
        for (; steps < 3 && lhs < rhs; ++steps) lhs *= 200;
        if (steps > more) more = steps;
    }
    const int c = kModCount[S - kModSlicesLo] + more;
    return c < kMaxMods ? c : kMaxMods;
}
// Capacity (moduli) a purification of n levels with S slices may use, by either
// method and at any occupation (one level needs the most), and at any n: 0 for
// digit slices.
constexpr int mod_capacity(int S, int n) { return mod_count(S, n, 1, true); }
constexpr int mod_capacity(int S) { return mod_capacity(S, 1 << 24); }
// Moduli of the adjoint's backward products, whose operands Y and Y P have no
// bound on their row norms but sqrt(n) times the row maximum.  Two moduli more
// leave about n 2^-58.4 m_i m_j (S = 7; S = 6 n 2^-50.8) where the slices drop 2^-48
// (2^-40) sqrt(n) m_i m_j.  Gradients against 11 slices, n = 1400 .. 3000, error
// over that with S slices: 0.02 (S = 6) and 0.13 (S = 7), geometric means; S = 8
// and its 16 moduli FP64 rounding, as with slices.
constexpr int mod_backward(int S) {
    if (S < kModSlicesLo || S > kModSlicesHi) return 0;
    const int c = kModCount[S - kModSlicesLo] + 2;
    return c < kMaxMods ? c : kMaxMods;
}

// Reconstruction constants of N moduli.  C' = X Y mod M satisfies C' / M =
// frac(sum_m u_m y_m / p_m) for any representative u_m of its residue, y_m =
// (M / p_m)^-1 mod p_m.  y_m / p_m is kept as w0 2^-40 + w1 2^-80 with
// integers w0, w1 <= 2^40, so the sums over u_m in [0, 255] are exact in
// FP64 (255 x 16 x 2^40 < 2^53) and the fraction is off by less than
// 255 N 2^-81 < 2^-69.
struct CrtTable {
    double w0[kMaxMods], w1[kMaxMods];
    double k0, k1;        // 128 sum w0, 128 sum w1 (bytes are stored as u + 128)
    double mh, ml;        // M 2^-80 as a double and its remainder
    double limit;         // largest admissible row norm of X: sqrt(M / 2), a little less
};

constexpr int inverse_mod(int a, int p) {
    for (int x = 1; x < p; ++x)
        if ((a * x) % p == 1) return x;
    return 0;
}

constexpr double pow2(int e) {
    double v = 1.0;
    for (int i = 0; i < (e < 0 ? -e : e); ++i) v = e < 0 ? v * 0.5 : v * 2.0;
    return v;
}

constexpr CrtTable make_crt(int N) {
    CrtTable t{};
    unsigned __int128 M = 1;
    for (int m = 0; m < N; ++m) M *= unsigned(kMods[m]);
    double s0 = 0.0, s1 = 0.0;
    for (int m = 0; m < N; ++m) {
        const int p = kMods[m];
        int rest = 1;
        for (int q = 0; q < N; ++q)
            if (q != m) rest = int((int64_t(rest) * kMods[q]) % p);
        const uint64_t y = uint64_t(inverse_mod(rest, p));
        const uint64_t a = y << 40;
        const uint64_t hi = a / uint64_t(p), rem = a % uint64_t(p);
        const uint64_t lo = ((rem << 40) + uint64_t(p) / 2) / uint64_t(p);
        t.w0[m] = double(hi);
        t.w1[m] = double(lo);
        s0 += t.w0[m];
        s1 += t.w1[m];
    }
    t.k0 = 128.0 * s0;
    t.k1 = 128.0 * s1;
    const double md = double(M);                  // nearest double
    const double rem = md >= double(M) && (unsigned __int128)(md) > M
                           ? -double((unsigned __int128)(md) - M)
                           : double(M - (unsigned __int128)(md));
    t.mh = md * pow2(-80);
    t.ml = rem * pow2(-80);
    // sqrt(M / 2) by Newton's iteration, less 2^-13 of it
    const double half = md * 0.5;
    double r = pow2(60);
    for (int i = 0; i < 60; ++i) r = 0.5 * (r + half / r);
    t.limit = r * (1.0 - 0x1p-13);
    return t;
}

template <int N>
struct Crt {
    static constexpr CrtTable table = make_crt(N);
};

// The limit for N moduli (kModMin .. kMaxMods).
inline double crt_limit(int N) {
    static constexpr double limits[kMaxMods - kModMin + 1] = {
        Crt<11>::table.limit, Crt<12>::table.limit, Crt<13>::table.limit,
        Crt<14>::table.limit, Crt<15>::table.limit, Crt<16>::table.limit};
    return limits[N - kModMin];
}

}  // namespace dmp
