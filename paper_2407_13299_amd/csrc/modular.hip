// Residue products (see modular.hpp): for every modulus p_m the INT8 or FP16
// matrix product of the operands' residue planes, reduced modulo p_m and
// stored as bytes (k_residue_gemm); then the combination to FP64 and the
// product's epilogue (k_combine).
#include <type_traits>
#include <vector>

#include "coef.hpp"
#include "host.hpp"
#include "ldsload.hpp"
#include "residues.hpp"

namespace dmp {

struct ModRow {
    int p, c16;       // modulus, 2^16 mod p
    float inv;        // 1 / p
};
struct ModRows {
    ModRow r[kMaxMods];
};
constexpr ModRows make_rows() {
    ModRows t{};
    for (int m = 0; m < kMaxMods; ++m) t.r[m] = ModRow{kMods[m], 65536 % kMods[m], 1.0f / float(kMods[m])};
    return t;
}
__constant__ const ModRows kModRows = make_rows();

struct CrtTables {
    CrtTable t[kMaxMods - kModMin + 1];
};
constexpr CrtTables make_crts() {
    return CrtTables{{Crt<11>::table, Crt<12>::table, Crt<13>::table, Crt<14>::table, Crt<15>::table, Crt<16>::table}};
}
__constant__ const CrtTables kCrtTables = make_crts();

// One workgroup of WM x WN wavefronts owns a tile of 16 WM FM rows x 16 WN FN
// columns of one modulus' product; each wavefront FM x FN blocks of 16 x 16,
// so a chunk (64 INT8 or 32 FP16 reduction elements) takes FM FN matrix
// instructions on FM + FN fragments of 1 KiB read from LDS.
//
// Bound: the chip's power limit under the matrix cores' load (residues are
// dense random bytes; the clock falls to 1.7 GHz) and, behind it, the LDS,
// which serves 128 bytes a cycle: unlike the slice GEMM, where S (S + 1) / 2
// products share 2 S fragments, every product here reads its own.  Hence
// 256 x 256 tiles of 8 wavefronts, 128 x 64 each (12 fragments read per 32
// products, 128 accumulator registers, two wavefronts per SIMD, one
// workgroup per CU).  16 x 16 x 64 products in boustrophedon order (one
// operand changes from product to product) need less power than 32 x 32 x 32
// ones: at n = 8192, 13 moduli on random residues, 2.64 against 2.86 ms
// (2.71 and 2.50 POP/s at 1.72 and 1.50 GHz); row order 2.70 ms.  128 x 256
// tiles, two workgroups per CU: 3.2 ms; all reads of a chunk ahead of its
// products: 3.1 ms.
//
// Pipeline: fragments go from memory straight into LDS, NBUF stages of one
// chunk, NBUF - 1 chunks ahead.  The fragments of chunk c + 1 are read from
// LDS into registers between the products of chunk c, one read or load after
// each product, so that neither the LDS latency, nor the barrier, nor a run
// of other instructions stands between two products.  At the end of chunk c a
// wavefront waits for its own loads of chunk c + 2 and the barrier publishes
// that chunk; the stage reloaded during chunk c held chunk c - 1, whose
// fragment reads had returned before the products of chunk c - 1 were
// issued, ahead of that barrier.
//
// The accumulators start at a multiple of p above K 2^14 (INT8), so every
// sum is positive: x mod p from its 16-bit halves, z = lo + hi (2^16 mod p)
// < 2^22, q = rint(z / p) in FP32 (off by less than 2^-9.4, closer than any
// z / p comes to a tie for odd p), r = z - q p.  FP16 sums are exact in FP32
// up to 2^24, so they are reduced every 31 chunks.
template <bool FP16, int WM, int WN, int FM, int FN, int NBUF, int OCC>
__global__ __launch_bounds__(64 * WM * WN, OCC) void k_residue_gemm(GemmParams p, int upper, CoefArgs extra) {
    constexpr int WAVES = WM * WN;
    constexpr int AB = WM * FM, BB = WN * FN;       // 16-row blocks of the tile
    constexpr int BLOCKS = AB + BB;                 // fragments of a stage
    constexpr int STAGE = BLOCKS * kFragBytes;
    constexpr int PER = BLOCKS / WAVES;             // loads per wavefront and stage
    static_assert(BLOCKS % WAVES == 0 && NBUF >= 4 && FM % 2 == 0 && FN % 2 == 0,
                  "equal loads per wavefront, whole 32 x 32 blocks");
    __shared__ __align__(16) uint8_t lds[NBUF][STAGE];

    if (int(blockIdx.x) < extra.count) {
        if (threadIdx.x < 256) coef_block(extra, reinterpret_cast<double*>(&lds[0][0]));
        return;
    }
    const int b = int(blockIdx.x) - extra.count;
    const int nb = int(gridDim.x) - extra.count;
    const int xcd = b & 7, qq = nb >> 3, rem = nb & 7, loc = b >> 3;
    const int t = p.spread ? b : (xcd < rem) ? xcd * (qq + 1) + loc : rem * (qq + 1) + (xcd - rem) * qq + loc;
    const Tile tile = p.mtiles[t];
    const int mod = int(tile.mat >> 24), mat = p.lone ? 0 : int(tile.mat & 0xffffffu);
    const MatDesc d = p.descs ? p.descs[mat] : p.one;
    const DevState* st = p.states ? p.states + mat : nullptr;
    if (st != nullptr && st->done) return;
    // the exponents of the output's planes, which the combination forms: each
    // row's once, by the first modulus' diagonal tiles (in the combination every
    // wavefront would work them out again, a tenth of its instructions: n =
    // 2048 36 and 30 against 34 and 28 us), behind the first loads
    auto exponents = [&]() __attribute__((always_inline)) {
        constexpr int ROWS = 16 * WM * FM;
        const int row = int(tile.I) * ROWS + int(threadIdx.x);
        if (d.expo_out != nullptr && mod == 0 && tile.I == tile.J && int(threadIdx.x) < ROWS &&
            row < int(round_up(d.M, kPad))) {
            d.expo_out[row] = residue_exponent(d.maxin[row], d.KC * (FP16 ? 16 : 32), kLamIterate, d.limit);
            if (d.clear != nullptr) d.clear[row] = 0;
        }
    };
    if (st != nullptr && p.skip_zero && st->gamma == 0.0) {
        exponents();
        return;
    }
    const bool clocked = p.clk != nullptr;
    const uint64_t clk_c = clocked ? __builtin_amdgcn_s_memtime() : 0;
    const uint64_t clk_r = clocked ? __builtin_amdgcn_s_memrealtime() : 0;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // wavefronts w and w + 4 share a SIMD: the lower half of the tile's
    // wavefronts is rotated against the upper one, so that a tile of which
    // only the left or only the upper half is in the matrix keeps every SIMD
    // busy with one wavefront
    const int wm = wave / WN, wn = (wave % WN + wm * (WN / 2)) % WN;
    const int rbs = int(round_up(d.M, kPad)) / 16, cbs = int(round_up(d.N, kPad)) / 16;
    const int RC = __builtin_amdgcn_readfirstlane(d.KC) / 2;   // chunks
    const int64_t a_rb = d.a_rb_stride, b_rb = d.b_rb_stride;
    const uint8_t* pa = d.pa + int64_t(mod) * rbs * a_rb;
    const uint8_t* pb = d.pb + int64_t(mod) * cbs * b_rb;

    // fragment f of a stage: 16-row block f of the left operand's part of the
    // tile, then of the right's; blocks past the operand's last (a tile
    // reaching beyond the padded matrix) load the last one and are not stored
    v4i dsc[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int f = wave * PER + i;
        const uint8_t* base;
        int64_t bytes;
        if (f < AB) {
            base = pa + int64_t(min(int(tile.I) * AB + f, rbs - 1)) * a_rb;
            bytes = a_rb;
        } else {
            base = pb + int64_t(min(int(tile.J) * BB + f - AB, cbs - 1)) * b_rb;
            bytes = b_rb;
        }
        dsc[i] = sgpr_desc(base, int(bytes));
    }
    const uint32_t lbase = lds_offset(&lds[0][0]) + uint32_t(wave * PER * kFragBytes);
    // load number i of chunk c into LDS stage ``slot``
    auto load = [&](int i, int c, int slot) __attribute__((always_inline)) {
        frag_to_lds(dsc[i], lbase + uint32_t(slot * STAGE + i * kFragBytes), lane * 16, c * kFragBytes);
    };
    auto issue = [&](int c, int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < PER; ++i) load(i, c, slot);
    };

    using Acc = typename std::conditional<FP16, v4f, v4i>::type;
    const ModRow mr = kModRows.r[mod];
    const int pm = mr.p;
    Acc acc[FM][FN];
    {
        using E = typename std::conditional<FP16, float, int>::type;
        const E bias = FP16 ? E(0) : E((RC * (64 << 14) / pm + 1) * pm);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[i][j] = Acc{bias, bias, bias, bias};
    }

    struct Frags {
        v4i a[FM], b[FN];
    };
    // fragment number i (left operand's first) of the chunk in stage ``slot``
    auto read = [&](int i, int slot, Frags& f) __attribute__((always_inline)) {
        const uint8_t* s = &lds[0][0] + slot * STAGE + lane * 16;
        if (i < FM)
            f.a[i] = *reinterpret_cast<const v4i*>(s + (wm * FM + i) * kFragBytes);
        else
            f.b[i - FM] = *reinterpret_cast<const v4i*>(s + (AB + wn * FN + i - FM) * kFragBytes);
    };
    const float inv = mr.inv, pf = float(pm);
    // FP32 integers |x| <= 2^24 to |x| <= p / 2: the first quotient may be
    // off by one, the second, of a number below 2 p, is exact
    auto fold = [&](float x) __attribute__((always_inline)) {
        x = __builtin_fmaf(-rintf(x * inv), pf, x);
        return __builtin_fmaf(-rintf(x * inv), pf, x);
    };

#pragma unroll
    for (int s = 0; s < NBUF - 1; ++s)
        if (s < RC) issue(s, s);
    exponents();
    if (RC >= NBUF - 1) ops_wait<(NBUF - 3) * PER>(); else ops_wait<0>();
    bare_barrier();
    Frags fr[2];
#pragma unroll
    for (int i = 0; i < FM + FN; ++i) read(i, 0, fr[0]);
    int slot = 0, flush = 0;
    // one chunk: its products, with the fragment reads of the next chunk and
    // the loads of chunk c + NBUF - 1 (MORE) spread between them.  After the
    // last chunk the reads are of a stage whose contents are not used (no
    // branch may stand between reads and products: the compiler would wait
    // for every read at once).
    auto step = [&](int c, const Frags& cur, Frags& nxt, auto more) __attribute__((always_inline)) {
        constexpr bool MORE = decltype(more)::value;
        constexpr int R = FM + FN, OPS = R + (MORE ? PER : 0), Q = FM * FN;
        const int prev = slot == 0 ? NBUF - 1 : slot - 1;
        const int next = slot == NBUF - 1 ? 0 : slot + 1;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int i = q / FN, j = (i & 1) ? FN - 1 - q % FN : q % FN;
            if constexpr (FP16)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                    __builtin_bit_cast(v8h, cur.a[i]), __builtin_bit_cast(v8h, cur.b[j]), acc[i][j], 0, 0, 0);
            else
                acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(cur.a[i], cur.b[j], acc[i][j], 0, 0, 0);
#pragma unroll
            for (int o = q * OPS / Q; o < (q + 1) * OPS / Q; ++o) {
                if (o < R) read(o, next, nxt);
                else load(o - R, c + NBUF - 1, prev);
            }
            if (q & 1) __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_sched_barrier(0);
        vm_wait<MORE ? (NBUF - 3) * PER : 0>();
        bare_barrier();
        slot = next;
        if constexpr (FP16) {
            if (++flush == 31) {
                flush = 0;
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j)
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[i][j][v] = fold(acc[i][j][v]);
            }
        }
    };
    // a wavefront whose blocks all lie outside the matrix (or below the
    // diagonal) only loads
    const int first_row = int(tile.I) * AB * 16 + wm * FM * 16, first_col = int(tile.J) * BB * 16 + wn * FN * 16;
    const bool idle = first_row >= d.M || first_col >= d.N || (upper && first_row >= first_col + FN * 16);
    if (__builtin_amdgcn_readfirstlane(int(idle))) {
        for (int c = 0; c < RC; ++c) {
            const bool more = c + NBUF - 1 < RC;
            if (more) issue(c + NBUF - 1, slot == 0 ? NBUF - 1 : slot - 1);
            if (more) vm_wait<(NBUF - 3) * PER>(); else vm_wait<0>();
            bare_barrier();
            slot = slot == NBUF - 1 ? 0 : slot + 1;
        }
        return;
    }
    int c = 0;
    for (; c + NBUF < RC; c += 2) {
        step(c, fr[0], fr[1], std::true_type{});
        step(c + 1, fr[1], fr[0], std::true_type{});
    }
    for (; c < RC; c += 2) {
        if (c + NBUF - 1 < RC) issue(c + NBUF - 1, slot == 0 ? NBUF - 1 : slot - 1);
        step(c, fr[0], fr[1], std::false_type{});
        if (c + 1 < RC) step(c + 1, fr[1], fr[0], std::false_type{});
    }

    // ---- residues of the sums, u + 128 as bytes --------------------------------
    // in 32 x 32 blocks of 1 KiB: byte 16 L + v of a block is row (L / 32) 4 +
    // 8 (v / 4) + v % 4, column L % 32 (the order in which the combination's
    // wavefronts hold a quadrant).  Of a block's 2 x 2 matrix-instruction
    // results lane l holds column l % 16 and rows 4 (l / 16) .. + 3; exchanging
    // the right results of lanes 0 .. 31 with the left ones of lanes 32 .. 63
    // leaves every lane 16 bytes of one column.
    const int64_t plane = int64_t(rbs / 2) * (cbs / 2) * kFragBytes;
    uint8_t* out = d.res + int64_t(mod) * plane +
                   (((lane >> 4) & 1) * 32 + (lane >> 5) * 16 + (lane & 15)) * 16;
    const uint32_t neg = uint32_t(256 - pm);
    const uint32_t halves = 1u | (uint32_t(mr.c16) << 16);
    auto residue = [&](auto x) __attribute__((always_inline)) -> uint32_t {
        if constexpr (FP16) {
            return uint32_t(int(fold(x)));
        } else {
            typedef unsigned short us2 __attribute__((ext_vector_type(2)));
            const uint32_t z = __builtin_amdgcn_udot2(__builtin_bit_cast(us2, uint32_t(x)),
                                                      __builtin_bit_cast(us2, halves), 0u, false);
            // q in the low bits of q + 1.5 2^23; only the low byte of z - q p
            // is kept, so the bits above q do no harm
            const float q = __builtin_fmaf(float(z), inv, 12582912.0f);
            return z + __umul24(__float_as_uint(q), neg);
        }
    };
    auto pack = [&](const Acc& a) __attribute__((always_inline)) {
        uint32_t r[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = residue(a[e]);
        return (__builtin_amdgcn_perm(r[1], r[0], 0x0c0c0400u) | __builtin_amdgcn_perm(r[3], r[2], 0x04000c0cu)) ^
               0x80808080u;
    };
#pragma unroll
    for (int i = 0; i < FM; i += 2)
#pragma unroll
        for (int j = 0; j < FN; j += 2) {
            const int rb = (int(tile.I) * AB + wm * FM + i) / 2, cb = (int(tile.J) * BB + wn * FN + j) / 2;
            if (rb >= rbs / 2 || cb >= cbs / 2 || (upper && rb > cb)) continue;   // wave-uniform
            uint32_t w[4];
#pragma unroll
            for (int ti = 0; ti < 2; ++ti) {
                const auto sw = __builtin_amdgcn_permlane32_swap(pack(acc[i + ti][j]), pack(acc[i + ti][j + 1]),
                                                                 false, false);
                w[2 * ti] = sw[0];
                w[2 * ti + 1] = sw[1];
            }
            *reinterpret_cast<uint4*>(out + (int64_t(rb) * (cbs / 2) + cb) * kFragBytes) =
                make_uint4(w[0], w[1], w[2], w[3]);
        }
    if (clocked) {
        const uint64_t dc = __builtin_amdgcn_s_memtime() - clk_c;
        const uint64_t dr = __builtin_amdgcn_s_memrealtime() - clk_r;
        if (threadIdx.x == 0) {
            atomicAdd(p.clk + 0, static_cast<unsigned long long>(dc));
            atomicAdd(p.clk + 1, static_cast<unsigned long long>(dr));
        }
    }
}

// ---- combination ----------------------------------------------------------

template <class T>
using Global = __attribute__((address_space(1))) T;

// Sum over a wavefront: within rows of 16 lanes by data parallel primitives
// (no LDS), then the four rows.
__device__ inline double sum64(double v) {
    auto ror = [](double x, auto n) __attribute__((always_inline)) {
        const uint64_t b = static_cast<uint64_t>(__double_as_longlong(x));
        const uint32_t lo = uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(b)), 0x120 + decltype(n)::value, 0xf, 0xf, false));
        const uint32_t hi = uint32_t(__builtin_amdgcn_update_dpp(0, int(b >> 32), 0x120 + decltype(n)::value, 0xf, 0xf, false));
        return __longlong_as_double(static_cast<long long>((uint64_t(hi) << 32) | lo));
    };
    v += ror(v, std::integral_constant<int, 8>{});
    v += ror(v, std::integral_constant<int, 4>{});
    v += ror(v, std::integral_constant<int, 2>{});
    v += ror(v, std::integral_constant<int, 1>{});
    const uint64_t b = static_cast<uint64_t>(__double_as_longlong(v));
    auto row = [&](int r) __attribute__((always_inline)) {
        const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(b)), 16 * r));
        const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(b >> 32), 16 * r));
        return __longlong_as_double(static_cast<long long>((uint64_t(hi) << 32) | lo));
    };
    return (row(0) + row(1)) + (row(2) + row(3));
}

// Maxima over the 16 lanes of a row (data parallel primitives, no LDS).
__device__ inline uint32_t max16(uint32_t v) {
    auto ror = [](uint32_t x, auto n) __attribute__((always_inline)) {
        return uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x120 + decltype(n)::value, 0xf, 0xf, false));
    };
    v = max(v, ror(v, std::integral_constant<int, 8>{}));
    v = max(v, ror(v, std::integral_constant<int, 4>{}));
    v = max(v, ror(v, std::integral_constant<int, 2>{}));
    return max(v, ror(v, std::integral_constant<int, 1>{}));
}

constexpr bool pur_mode(int mode) {
    return mode == EPI_SQUARE || mode == EPI_UPDATE || mode == EPI_SQUARE_TRS4;
}

// Rebuilds C' = X Y from its residues (modular.hpp) and runs the FP64 end of
// the product, C = C' 2^(t_i + t_j), by mode as listed at the head of
// ozgemm.hip.  One workgroup per 32 x 64 tile of p.tiles, a quarter (WAVES = 8)
// or half (4) of one of its two 32 x 32 quadrants per wavefront: lane l holds
// column l % 32 and rows (l / 32) 4 + 8 g + e, e < 4, of one or two row groups
// g, the order in which the residues are stored.
//
// The purification modes then form the residues of the output from the tile
// in LDS: half of the wavefronts the fragments of its two 16-row blocks, half,
// transposed, those of its four 16-column blocks.  So an iterate or a square
// is split without being read again, and without the launch that did
// (k_residues: 23 us at n = 2048, 290 us at n = 8192).  The exponents come from
// the row maxima of the iterate before the product (MatDesc::limit), as the
// output's own are known only when every tile is done; the residue GEMM works
// them out.
//
// Bound: memory for many tiles (N to 2 N bytes of residues and 12 to 28 bytes
// of FP64 per element; n = 2048: 28 and 34 us) and instructions; for few tiles the chain of
// latencies, with one wavefront per SIMD (n = 256: 7.9 and 9.0 us, 4.5 of them
// the two rounds of loads and the launch).  Hence 8 wavefronts rather than 4
// (9.6 and 11 us) where the tiles do not fill the chip; loops and constants
// that need few instruction and scalar-cache lines (store_residues; n = 256
// as a whole 680 to 541 us); wavefront sums without LDS; every load issued before
// the first result is formed.  The partial sums are formed per row group and
// added in one order, so that both widths give the same bits.  Row maxima,
// which only choose powers of two, are kept to the upper word, rounded up.
// MIXED: the matrices of the batch have up to N moduli, each its own count
// (MatDesc::nmod), whose constants come from a table; beyond the count they are
// zero, so that a matrix gets the bits of a launch of its own.  One launch
// instead of one per count: a batch of 8 of n = 48 .. 100 1.06 -> 0.63 ms, 48 of
// 128 .. 512 at 30 % filling 5.8 -> 4.7 ms.
// (The update at 4 wavefronts needs 145 registers: three wavefronts per SIMD.)
template <int N, int MODE, bool FP16, int WAVES, bool MIXED>
__global__ __launch_bounds__(64 * WAVES, MODE == EPI_UPDATE && WAVES == 4 ? 3 : 4) void k_combine(GemmParams p) {
    constexpr bool PUR = pur_mode(MODE);
    constexpr bool UPPER = MODE != EPI_STORE;
    static_assert(WAVES == 8 || (WAVES == 4 && !FP16), "a lane's part of the planes: 8 or 16 bytes");
    constexpr int G = 8 / WAVES, LDT = 65;
    __shared__ double red[8][kPartials];
    __shared__ double out_tile[PUR ? 32 * LDT : 1];
    const int b = blockIdx.x, nb = gridDim.x;
    const int xcd = b & 7, qq = nb >> 3, rem = nb & 7, loc = b >> 3;
    const int t = p.spread ? b : (xcd < rem) ? xcd * (qq + 1) + loc : rem * (qq + 1) + (xcd - rem) * qq + loc;
    const Tile tile = p.tiles[t];
    const int mat = p.lone ? 0 : int(tile.mat);
    const MatDesc d = p.descs ? p.descs[mat] : p.one;
    const DevState* st = p.states ? p.states + mat : nullptr;
    if (st != nullptr && st->done) return;
    const int mods = MIXED ? __builtin_amdgcn_readfirstlane(d.nmod) : N;
    double alpha = 0.0, beta = 0.0, gamma = 1.0;
    if constexpr (MODE == EPI_UPDATE) {
        alpha = st->alpha;
        beta = st->beta;
        gamma = st->gamma;
    }
    const bool has_product = MODE != EPI_UPDATE || !p.skip_zero || gamma != 0.0;   // a TRS4 step without one
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    // quadrant ``quad`` of the tile, row groups g0 .. g0 + G - 1 of it
    const int quad = wave / (4 / G), g0 = wave % (4 / G) * G;
    const int qr = int(tile.I), qc = 2 * int(tile.J) + quad;
    const int M = __builtin_amdgcn_readfirstlane(d.M), NC = __builtin_amdgcn_readfirstlane(d.N);
    const int ldc = __builtin_amdgcn_readfirstlane(d.ldc);
    const int lrow = (lane >> 5) * 4, lcol = lane & 31;
    double s0[G] = {}, s1[G] = {};
    // the planes of the output (below): what this wavefront writes, and the
    // exponent of the lane's row
    constexpr int K64 = FP16 ? 2 : 1;             // fragments per 64 reduction elements
    const int half = int(tile.I) & 1;
    const bool diag = int(tile.I) >> 1 == int(tile.J), rows = wave < WAVES / 2;
    constexpr int NE = WAVES == 8 ? 8 : 16;       // elements per lane
    const int lr = WAVES == 8 ? (rows ? wave >> 1 : wave - 4) * 16 + (lane & 15)
                              : (rows ? wave * 16 : (wave - 2) * 32 + (lane >> 5) * 16) + (lane & 15);
    const int k0 = WAVES == 8 ? (rows ? (wave & 1) * 32 : 0) + (lane >> 4) * 8
                              : (rows ? lane >> 4 : (lane >> 4) & 1) * 16;
    const int row = rows ? 32 * int(tile.I) + lr : 64 * int(tile.J) + lr;
    const int tx = PUR ? d.expo_out[row] : 0;
    ModSplit split{};
    if constexpr (PUR) split = lane_split();

    auto quadrant = [&](auto full) __attribute__((always_inline)) {
        constexpr bool FULL = decltype(full)::value;
        const int cbs = int(round_up(NC, kPad)) / 32;
        const int64_t plane = int64_t(round_up(M, kPad) * round_up(NC, kPad));
        using Word = typename std::conditional<G == 4, v4i, typename std::conditional<G == 2, v2i, v1i>::type>::type;
        Word w[N];
        if (has_product) {
            const Global<Word>* src = reinterpret_cast<const Global<Word>*>(
                reinterpret_cast<uint64_t>(d.res) + (int64_t(qr) * cbs + qc) * kFragBytes + 4 * g0);
#pragma unroll
            for (int m = 0; m < N; ++m)
                w[m] = src[((MIXED ? min(m, mods - 1) : m) * plane + lane * 16) / int(sizeof(Word))];
        }
        // exponents: rows in groups of four
        const Global<v4i>* ea = reinterpret_cast<const Global<v4i>*>(reinterpret_cast<uint64_t>(d.ea + qr * 32 + 8 * g0 + lrow));
        v4i er[G];
#pragma unroll
        for (int g = 0; g < G; ++g) er[g] = ea[2 * g];
        const int fj = reinterpret_cast<const Global<int>*>(reinterpret_cast<uint64_t>(d.eb))[qc * 32 + lcol];
        // element v of the quadrant: in the matrix (and, for the modes on one
        // triangle, on or above the diagonal)
        const int row0 = qr * 32 + 8 * g0 + lrow, col = qc * 32 + lcol;
        auto inside = [&](int v) __attribute__((always_inline)) {
            const int row = row0 + 8 * (v >> 2) + (v & 3);
            return FULL || (row < M && col < NC && (!UPPER || row <= col));
        };
        const int voff = lrow * ldc + lcol;
        auto at = [&](const double* base, int v) __attribute__((always_inline)) {
            // wave-uniform part of the address apart from the lane's
            return reinterpret_cast<Global<double>*>(
                reinterpret_cast<uint64_t>(base) +
                8 * (int64_t(qr * 32 + 8 * (g0 + (v >> 2)) + (v & 3)) * ldc + qc * 32));
        };
        double pv[4 * G], xv[4 * G], hv[4 * G];
        // a matrix with weight zero is not read (the canonical branch c >= 1/2
        // has alpha = 0, a TRS4 step with a product alpha = beta = 0)
        auto fetch = [&](const double* src, bool wanted, double (&to)[4 * G]) __attribute__((always_inline)) {
#pragma unroll
            for (int v = 0; v < 4 * G; ++v) to[v] = 0.0;
            if (wanted) {
#pragma unroll
                for (int v = 0; v < 4 * G; ++v)
                    if (inside(v)) to[v] = at(src, v)[voff];
            }
        };
        if constexpr (PUR) fetch(d.P, MODE != EPI_UPDATE || alpha != 0.0, pv);
        if constexpr (MODE == EPI_UPDATE) {
            fetch(d.X2, beta != 0.0, xv);
            fetch(d.H, true, hv);
        }
        uint32_t hi[4 * G], cmax = 0;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            double out4[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int v = 4 * g + e;
                const int row = row0 + 8 * g + e;
                double c = 0.0;
                if (has_product) {
                    // the fraction C' / M as f0 2^-40 + f1 2^-80 less its
                    // nearest integer, times M
                    const CrtTable& T = MIXED ? kCrtTables.t[mods - kModMin] : Crt<N>::table;
                    double f0 = -T.k0, f1 = -T.k1;
#pragma unroll
                    for (int m = 0; m < N; ++m) {
                        const double u = double((uint32_t(w[m][g]) >> (8 * e)) & 0xffu);
                        f0 = __builtin_fma(u, T.w0[m], f0);
                        f1 = __builtin_fma(u, T.w1[m], f1);
                    }
                    const double k = rint(__builtin_fma(f1, 0x1p-80, f0 * 0x1p-40));
                    const double x = __builtin_fma(__builtin_fma(k, -0x1p40, f0), 0x1p40, f1);
                    const int ei = er[g][e];
                    c = ldexp(__builtin_fma(x, T.mh, x * T.ml), ei + fj);
                    if (ei >= kNonFiniteExp || fj >= kNonFiniteExp) c = __builtin_nan("");
                }
                double o = c;
                if constexpr (PUR) {
                    const bool diag = !FULL && row == col;
                    const double mult = diag ? 1.0 : 2.0;
                    const double pij = pv[v];
                    if (inside(v)) {
                        if constexpr (MODE == EPI_SQUARE) {
                            if (diag) s0[g] += pij - c;
                            s1[g] += mult * c * ((diag ? 1.0 : 0.0) - pij);
                        } else if constexpr (MODE == EPI_SQUARE_TRS4) {
                            const double r = pij - c;
                            s0[g] += mult * c * (4.0 * pij - 3.0 * c);
                            s1[g] += mult * r * r;
                        } else {
                            o = alpha * pij + beta * xv[v] + gamma * c;
                            s0[g] += mult * o * hv[v];
                            if (diag) s1[g] += o;
                        }
                    }
                }
                out4[e] = o;
                if constexpr (PUR)
                    out_tile[(8 * (g0 + g) + lrow + e) * LDT + quad * 32 + lcol] = inside(v) ? o : 0.0;
                const uint32_t h = uint32_t(static_cast<uint64_t>(__double_as_longlong(o)) >> 32) & 0x7fffffffu;
                hi[v] = inside(v) ? h : 0u;
                cmax = max(cmax, hi[v]);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (inside(4 * g + e)) at(d.out, 4 * g + e)[voff] = out4[e];
            if (UPPER && !(PUR && p.upper_only)) {
                // the mirror: four consecutive elements of row ``col``
                Global<double>* mir = reinterpret_cast<Global<double>*>(
                    reinterpret_cast<uint64_t>(d.out) + 8 * (int64_t(col) * ldc + row0 + 8 * g));
                if constexpr (FULL) {
                    typedef double d2 __attribute__((ext_vector_type(2), aligned(8)));
                    Global<d2>* m2 = reinterpret_cast<Global<d2>*>(mir);
                    m2[0] = d2{out4[0], out4[1]};
                    m2[1] = d2{out4[2], out4[3]};
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (inside(4 * g + e) && row0 + 8 * g + e != col) mir[e] = out4[e];
                }
            }
        }
        // Row maxima (upper words).  Lanes 16 apart are combined two rows at
        // a time by an exchange, after which the even 16-lane rows hold the
        // first of the two rows and the odd ones the second; then over the
        // 16 lanes; lane k < 2 G of each 16-lane row holds pair k's maximum.
        auto word = [](uint32_t h) { return (uint64_t(h) << 32) | (h != 0 ? 0xffffffffu : 0u); };
        if (d.rowmax != nullptr) {
            uint32_t mine = 0;
#pragma unroll
            for (int k = 0; k < 2 * G; ++k) {
                const auto sw = __builtin_amdgcn_permlane16_swap(hi[2 * k], hi[2 * k + 1], false, false);
                const uint32_t m = max16(max(uint32_t(sw[0]), uint32_t(sw[1])));
                mine = (lane & 15) == k ? m : mine;
            }
            const int v = 2 * (lane & 15) + ((lane >> 4) & 1);
            if ((lane & 15) < 2 * G && mine != 0)
                atomicMax(reinterpret_cast<unsigned long long*>(d.rowmax) + row0 + 8 * (v >> 2) + (v & 3),
                          static_cast<unsigned long long>(word(mine)));
        }
        uint64_t* const cdst = UPPER ? d.rowmax : d.colmax;
        if (cdst != nullptr) {
            const auto sw = __builtin_amdgcn_permlane32_swap(cmax, cmax, false, false);
            const uint32_t m = max(uint32_t(sw[0]), uint32_t(sw[1]));
            if (lane < 32 && m != 0)
                atomicMax(reinterpret_cast<unsigned long long*>(cdst) + col, static_cast<unsigned long long>(word(m)));
        }
    };
    if (!UPPER || qr <= qc) {
        if ((!UPPER || qr < qc) && (qr + 1) * 32 <= M && (qc + 1) * 32 <= NC)
            quadrant(std::true_type{});
        else
            quadrant(std::false_type{});
    }
    if constexpr (PUR) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const double t0 = sum64(s0[g]), t1 = sum64(s1[g]);
            if (lane == 0) {
                red[wave * G + g][0] = t0;
                red[wave * G + g][1] = t1;
            }
        }
        __syncthreads();
        if (threadIdx.x < kPartials) {
            double r = 0.0;
#pragma unroll
            for (int i = 0; i < 8; ++i) r += red[i][threadIdx.x];
            p.partials[int64_t(t) * kPartials + threadIdx.x] = r;
        }

        // ---- residue planes of the output ------------------------------------
        // Rows (wave 0, 1): 16-row block ``wave`` of the tile over all 64
        // columns.  Columns (wave 2, 3): the mirror's rows, 16-column blocks 2
        // (wave - 2) and the next, lanes 0 .. 31 and 32 .. 63, over the tile's 32
        // rows.  On the diagonal the upper tile (I even) writes its rows
        // whole and the mirror of its right half, the lower one (I odd, whose
        // left half lies below the diagonal) the right half of its rows.
        if (diag && !rows && (half == 1 || wave < WAVES * 3 / 4)) return;
        const bool wanted = !diag || !rows || half == 0 || k0 >= 32;
        if (WAVES == 8 && !wanted) return;
        const int rbs = int(round_up(M, kPad)) / 16, RC = __builtin_amdgcn_readfirstlane(d.KC) / 2;
        const int64_t plane = int64_t(rbs) * RC * kFragBytes;
        // the lane's first element: reduction element ``pos`` of the chunk
        const int pos = rows ? k0 : half * 32 + k0;
        const int chunk = rows ? int(tile.J) : int(tile.I) >> 1;
        uint8_t* const at = d.planes_out + (int64_t(row / 16) * RC + chunk * K64) * kFragBytes +
                            (FP16 ? pos / 32 * kFragBytes + (pos % 32 / 8 * 16 + (lane & 15)) * 16
                                  : (pos / 16 * 16 + (lane & 15)) * 16 + pos % 16);
        double x[NE];
        if (rows) {
            // below the diagonal of a quadrant on it (the left one of an
            // upper tile, the right one of a lower one): the mirror's element
            const int c0 = half * 32;
            const bool on = diag && (k0 & 32) == c0;
#pragma unroll
            for (int i = 0; i < NE; ++i)
                x[i] = out_tile[on && lr > k0 - c0 + i ? (k0 - c0 + i) * LDT + c0 + lr : lr * LDT + k0 + i];
        } else {
#pragma unroll
            for (int i = 0; i < NE; ++i) x[i] = out_tile[(k0 + i) * LDT + lr];
        }
        store_residues<FP16>(x, tx, split, at, plane, mods, wanted);
    }
}

// Tiles from which a tile has 4 wavefronts instead of 8 (half the exponents,
// row maxima and requests per element).  Square and update, 4 and 8: 24
// matrices of n = 256 .. 1024, 2700 tiles, 61 and 76 against 72 and 83 us; n =
// 2048, 1056 tiles, 28.8 and 35.5 against 30.4 and 36.1 us; n = 1400, 506 tiles,
// square 17.6 against 16.5 us; n = 256, 20 tiles, 9.6 against 7.9 us.
constexpr int kFourWaveTiles = 1024;

template <int N, int MODE, bool MIXED>
static void combine_as(bool fp16, const GemmParams& p, int nout, hipStream_t stream) {
    if constexpr (pur_mode(MODE)) {
        if (fp16) {
            k_combine<N, MODE, true, 8, MIXED><<<nout, 512, 0, stream>>>(p);
            return;
        }
    }
    if (nout >= kFourWaveTiles)
        k_combine<N, MODE, false, 4, MIXED><<<nout, 256, 0, stream>>>(p);
    else
        k_combine<N, MODE, false, 8, MIXED><<<nout, 512, 0, stream>>>(p);
}

template <int N, int MODE>
static void combine(bool fp16, const GemmParams& p, int nout, hipStream_t stream) {
    if constexpr (pur_mode(MODE) && N > kModMin) {
        if (p.mixed) {
            combine_as<N, MODE, true>(fp16, p, nout, stream);
            return;
        }
    }
    combine_as<N, MODE, false>(fp16, p, nout, stream);
}

template <int N>
static int launch_combine(bool fp16, const GemmParams& p, int nout, hipStream_t stream) {
    switch (p.mode) {
        case EPI_STORE: combine<N, EPI_STORE>(fp16, p, nout, stream); break;
        case EPI_STORE_SYM: combine<N, EPI_STORE_SYM>(fp16, p, nout, stream); break;
        case EPI_SQUARE: combine<N, EPI_SQUARE>(fp16, p, nout, stream); break;
        case EPI_UPDATE: combine<N, EPI_UPDATE>(fp16, p, nout, stream); break;
        default: combine<N, EPI_SQUARE_TRS4>(fp16, p, nout, stream);
    }
    DMP_CHECK_HIP(hipGetLastError());
    return DMP_OK;
}

int launch_residue_gemm(dmp_kind kind, int nmod, int shape, const GemmParams& p, int ntiles, int nout,
                        hipStream_t stream, const CoefArgs& step) {
    if (ntiles <= 0 || nout <= 0) return DMP_OK;
    if ((kind != DMP_OZ_INT8 && kind != DMP_OZ_FP16) || nmod < kModMin || nmod > kMaxMods ||
        p.mtiles == nullptr || p.fix != nullptr || (p.mixed && (!pur_mode(p.mode) || nmod == kModMin))) {
        set_error("invalid residue product (%d moduli)", nmod);
        return DMP_EINVAL;
    }
    const int upper = p.mode == EPI_STORE ? 0 : 1;
    const int grid = ntiles + step.count;
    if (kind == DMP_OZ_FP16 && shape == kShapeWide)
        k_residue_gemm<true, 2, 4, 8, 4, 4, 2><<<grid, 512, 0, stream>>>(p, upper, step);
    else if (kind == DMP_OZ_FP16)
        k_residue_gemm<true, 2, 4, 4, 2, 4, 4><<<grid, 512, 0, stream>>>(p, upper, step);
    else if (shape == kShapeWide)
        k_residue_gemm<false, 2, 4, 8, 4, 4, 2><<<grid, 512, 0, stream>>>(p, upper, step);
    else
        k_residue_gemm<false, 2, 4, 4, 2, 4, 4><<<grid, 512, 0, stream>>>(p, upper, step);
    DMP_CHECK_HIP(hipGetLastError());
    static int (*const combine[kMaxMods - kModMin + 1])(bool, const GemmParams&, int, hipStream_t) = {
        launch_combine<11>, launch_combine<12>, launch_combine<13>,
        launch_combine<14>, launch_combine<15>, launch_combine<16>};
    return combine[nmod - kModMin](kind == DMP_OZ_FP16, p, nout, stream);
}

}  // namespace dmp
