// Device code shared by the residue split and the residue combination: the
// power of two of an operand row and the residues of its elements.
#pragma once

#include <hip/hip_fp16.h>

#include "common.hpp"

namespace dmp {

// Exponent t of an operand row of a residue product: X = rint(a 2^-t) with
// 2^-t the largest power of two that keeps the row norm of X within
// ``limit``.  The norm is bounded from the row maximum m (its bit pattern; only
// the upper word counts, rounded up): it is at most sqrt(K) m, and at most
// sqrt(lam m) for a positive semidefinite source with eigenvalues up to lam
// (|row i|^2 = (A^2)_ii <= lam A_ii <= lam m).
__device__ inline int residue_exponent(uint64_t bits, int K, double lam, double limit) {
    if (bits >= 0x7ff0000000000000ull) return kNonFiniteExp;
    if (bits == 0) return 0;
    const double m = __longlong_as_double(static_cast<long long>(bits | 0xffffffffull));
    double nu = sqrt(double(K)) * m;
    if (lam > 0.0) nu = fmin(nu, sqrt(lam * m));
    int en = 0, el = 0;
    const double fn = frexp(nu, &en), fl = frexp(limit, &el);
    return en - el + (fn > fl ? 1 : 0);
}

// Per modulus: 1 / p, 2^27 mod p (balanced) and 256 - p.  A wavefront holds
// them in its lanes, modulus m in lane m, from one load early on: read one
// modulus after another from memory they cost a scalar-cache miss every few.
struct alignas(16) ModSplit {
    double inv;
    int c;
    uint32_t neg;
};
struct ModSplits {
    ModSplit r[kMaxMods];
};
constexpr ModSplits make_splits() {
    ModSplits t{};
    for (int m = 0; m < kMaxMods; ++m) {
        const int p = kMods[m], c = (1 << 27) % p;
        t.r[m] = ModSplit{1.0 / p, c > p / 2 ? c - p : c, uint32_t(256 - p)};
    }
    return t;
}
__constant__ const ModSplits kModSplits = make_splits();
__device__ inline ModSplit lane_split() { return kModSplits.r[threadIdx.x & (kMaxMods - 1)]; }

// One lane's bytes of a fragment in each of ``mods`` planes: the balanced residues
// of X = rint(v 2^-t) for NE elements (8 or 16; FP16: 8, as halves); plane m
// starts at m ``plane`` bytes from ``base`` (a lane that is not ``wanted``
// stores nothing).  Per element X = Xh 2^27 + Xl exactly; per modulus z = Xh
// (2^27 mod p) + Xl, q = rint(z / p) (|X| < 2^62.2 with 16 moduli, so |z| < 2^43 and
// the product with 1 / p is off by less than 2^-17, closer than any z / p, p odd,
// comes to a tie: 2^-9), and
// z - q p modulo 256 is the residue's byte (p = 256: +-128 are the same byte).
// The integers z and q are read from the low words of z + 1.5 2^52 and q + 1.5
// 2^52: four full-rate instructions per modulus.  The moduli are a loop: as
// straight-line code, run once, they wait for instructions.
template <bool FP16, int NE>
__device__ __forceinline__ void store_residues(const double (&v)[NE], int t, const ModSplit& split, uint8_t* base,
                                               int64_t plane, int mods, bool wanted = true) {
    constexpr int E = FP16 ? 2 : 4, NW = NE / E;   // elements per word, words
    typedef uint32_t Words __attribute__((ext_vector_type(NW)));
    constexpr double kMagic = 0x1.8p52;
    auto low = [](double x) __attribute__((always_inline)) {
        return uint32_t(static_cast<uint64_t>(__double_as_longlong(x)));
    };
    double xh[NE], xl[NE];
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const double x = t >= kNonFiniteExp ? 0.0 : rint(ldexp(v[i], -t));
        xh[i] = rint(x * 0x1p-27);
        xl[i] = __builtin_fma(xh[i], -0x1p27, x);
    }
    const uint64_t invs = static_cast<uint64_t>(__double_as_longlong(split.inv));
#pragma unroll 1
    for (int m = 0; m < mods; ++m) {
        const double c = double(__builtin_amdgcn_readlane(split.c, m));
        const uint32_t neg = uint32_t(__builtin_amdgcn_readlane(int(split.neg), m));
        const double inv = __longlong_as_double(static_cast<long long>(
            (uint64_t(uint32_t(__builtin_amdgcn_readlane(int(invs >> 32), m))) << 32) |
            uint32_t(__builtin_amdgcn_readlane(int(uint32_t(invs)), m))));
        Words w;
#pragma unroll
        for (int g = 0; g < NW; ++g) {
            uint32_t b[E];
#pragma unroll
            for (int i = 0; i < E; ++i) {
                const double z = __builtin_fma(xh[g * E + i], c, xl[g * E + i]);
                const uint32_t q = low(__builtin_fma(z, inv, kMagic));
                // the low byte of z - q p (24-bit multiply-add: the bits
                // above do not matter)
                b[i] = low(z + kMagic) + __umul24(q, neg);
            }
            if constexpr (!FP16) {
                w[g] = __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u) |
                       __builtin_amdgcn_perm(b[3], b[2], 0x04000c0cu);
            } else {
                // balanced residues are exact FP16 values (|r| <= 128)
                uint32_t h = 0;
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    h |= uint32_t(__half_as_ushort(__int2half_rn(int(int8_t(uint8_t(b[i])))))) << (16 * i);
                w[g] = h;
            }
        }
        if (wanted) *reinterpret_cast<Words*>(base + m * plane) = w;
    }
}

}  // namespace dmp
