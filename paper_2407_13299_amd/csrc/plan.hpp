// Host-side planning of libdmp: tile orders, the split-tail plan, workspace
// carving, the grouping of a batch and the descriptors of every launch, and
// the caches the library keeps.  Pure C++17 (no HIP headers), so that this
// part also builds with a plain host compiler under the address, undefined
// behaviour and thread sanitizers (tests/host/).
#pragma once

#include <cstddef>
#include <cstdint>
#include <functional>
#include <list>
#include <map>
#include <memory>
#include <mutex>
#include <utility>
#include <vector>

#include "layout.hpp"

namespace dmp {

// Carves 256-byte-aligned regions out of a workspace; with base == nullptr it
// only measures.
class Carver {
public:
    explicit Carver(void* base) : base_(static_cast<uint8_t*>(base)) {}
    template <typename T>
    T* take(size_t count) {
        off_ = (off_ + 255) & ~size_t(255);
        T* p = base_ ? reinterpret_cast<T*>(base_ + off_) : nullptr;
        off_ += count * sizeof(T);
        return p;
    }
    size_t used() const { return (off_ + 255) & ~size_t(255); }

private:
    uint8_t* base_;
    size_t off_ = 0;
};

// ---- argument checks ------------------------------------------------------
int check_kind_slices(dmp_kind kind, int slices);
int validate_purify_args(const double* H, int n, int nocc, double tol, int max_iter,
                         const double* P);
int check_method_flags(int method, int flags);
// The caller's workspace starts on a 256-byte boundary (the carved regions
// are 256-byte aligned relative to it, and kernels load 16-byte vectors).
int check_workspace_alignment(const void* ws);

// ---- tile orders ----------------------------------------------------------
// Order of the TM x 64 output tiles of one matrix (TM = 128, or 64 for the
// 64-row variant): 512 x 512 super-tiles, row-major over super-tiles and
// within each; ``upper`` keeps the tiles that reach the upper triangle
// (column >= row somewhere in the tile).
void append_tiles(std::vector<Tile>& out, int tm, int tn, bool upper, uint32_t mat,
                  int TM = kTileM);
int tile_rows(int m, int TM = kTileM);
int tile_cols(int n);
int upper_tile_count(int n, int TM = kTileM);

// Tile list of the residue GEMM of an n x n product: all ``nmod`` moduli, one
// after the other (modulus in the top byte of ``mat``), tiles of shape
// ``shape`` in 1024 x 1024 super-tiles.
void append_residue_tiles(std::vector<Tile>& out, int n, int nmod, int shape, bool upper, uint32_t mat);
int residue_tile_count(int n, int shape, bool upper);   // per modulus
// Shape for a launch of the products of ``count`` matrices: 256 x 256 tiles
// where there are kWideTiles of them (all moduli) and they are not mostly
// empty.  A tile of a matrix costs its 64-element chunks and kTileStartChunks
// more; the chip does 2.8 small tiles in the time of a wide one.  One GEMM, wide
// and small: n = 700, 78 wide tiles, 12.2 and 11.6 us; n = 1024, 130 tiles, 16.1
// and 19.4 us; n = 1400 33.0 and 33.5 us; n = 2048 57 and 65 us; batches of 40 of
// n = 64 .. 256 (work in small tiles 2.2 times that in wide ones) 15.3 and
// 11.2 us, 48 of 128 .. 512 (2.6) 39.0 and 33.4 us, 30 of 100 .. 800 (2.8) 73.4
// and 73.9 us, 24 of 256 .. 1024 (2.9) 94.6 and 98.9 us.
constexpr int kWideTiles = 100, kTileStartChunks = 4, kSmallPerWide10 = 28;
int residue_shape(int count, const int* n, int nmod, bool upper);

// Workgroups ("units") of the split kernels for an operand of R rows.
int split_units_rowmax(int R);
int split_units_colmax(int R, int K);
int split_units_digits(int R, int KC);
int64_t chunks_of(int k, dmp_kind kind);
// Units of each stage of a set of operands; fills their first-unit fields.
struct SplitUnits {
    int rowmax = 0, colmax = 0, digits = 0;
};
void count_split_units(SplitDesc* d, int count, SplitUnits& u);
// Whether the digit split of a set takes the row maxima itself: every
// workgroup then reads its 32 rows over the whole reduction, instead of one or
// two launches before it.  That read is a chain of K / 64 loads: at K = 64 ..
// 512 the split takes 9 .. 11 us beside 5 us and two launches of 4 us, at K =
// 1301 60 us beside 12 + 11 us.  And where a row block has more than two
// workgroups (K above 256 in INT8, above 128 in FP16) it reads the operands
// again, from the caches, for each of them but one; beyond kSelfMaxBytes in all
// that costs more than the two launches, beyond kSelfMaxBytesRows more than the
// one of operands that are rows.  A whole product, launches and self: m x 64 x
// 512, m = 4096 (51 MB) 39 and 38 us, 8192 (101 MB) 45 and 50, 65536 242 and 279;
// rows alone, 2048 (25 MB) 32 and 32, 4096 36 and 39; batches, 24 of 64 .. 512 (61
// MB) 119 and 116, 16 of 256 .. 512 (99 MB) 105 and 111, FP16 24 of 64 .. 512 (156
// MB) 166 and 177; m x 64 x 256, 65536 131 and 124.
constexpr int kSelfMaxK = 512;
constexpr int64_t kSelfMaxBytes = 64000000, kSelfMaxBytesRows = 26000000;
bool split_takes_maxima(const SplitDesc* d, int count);

// ---- split tail -----------------------------------------------------------
// Tail split of ``ntiles`` tiles of equal cost: tiles [0, nfull) whole, the
// rest in nsplit parts each (nsplit == 1: no split).
struct TailSplit {
    int nfull, nsplit;
};
// ``slots`` workgroups run at once, so the tiles run in full rounds and a
// last round of r = ntiles mod slots tiles that leaves the rest of the chip
// idle; when there is at least one full round, those r tiles are split into
// as many parts as fill it (at most kMaxSplit, at least kMinSplitChunks of
// the ``min_kc`` chunks each, at most ``max_pieces`` parts in all).
TailSplit plan_tail_split(int ntiles, int slots, int min_kc, int max_pieces);
// The same for the tiles of one general product, which may also be too few to
// fill a quarter of the slots (half of the CUs): then every tile is split, if
// that shortens the reduction by at least kMinSavedChunks chunks (the fixup
// launch costs about 20 us: 4096 x 96 x 4096 at S = 8 298 -> 188 us, but 208
// tiles of 41 chunks in two parts 54 -> 77 us).
constexpr int kMinSavedChunks = 24;
TailSplit plan_gemm_split(int ntiles, int slots, int min_kc, int max_pieces);
// Tile height (32-row blocks) of a general m x n product, and of a batch of
// them: 64 rows, two workgroups per CU, below kLowTileCount tiles of 128 rows
// (one round of the chip; 1000 x 777 x 1301, 104 tiles: 60 -> 38 us).
constexpr int kLowTileCount = 256;
int gemm_tile_blocks(int m, int n, int S, dmp_kind kind);
int batch_tile_blocks(int count, const int* m, const int* n, int S, dmp_kind kind);
// Parts of a tail split a group of ``ntiles`` tiles of height 32 rb may need
// (the size of its part buffer in pieces, 0 when no split can arise).
int tail_split_capacity(int ntiles, int min_kc, int rb);

// ---- tuned choices --------------------------------------------------------
// Smallest slice count whose error model (fitted to measurements) meets
// ``target`` for an n x n purification.
int autotune_slices_model(int n, double target, dmp_kind kind);
// Slice count per matrix of a batch (slices > 0: that count for all).
void batch_slices(int count, const int* n, int slices, dmp_kind kind, std::vector<int>& s);
// Tile choice of the products of an n x n Ozaki purification (and of its
// adjoint): 32-row blocks per tile (2: 64-row tiles, 4: 128-row tiles) and
// whether the last, partly filled round of tiles is split along the
// reduction.  A function of (kind, S, n) only, from the measured table;
// ``forced_rb`` (2 or 4, 0 for none) overrides the height where it exists.
struct TileChoice {
    int rb;
    bool split_tail;
};
TileChoice tile_choice(dmp_kind kind, int S, int n, int forced_rb = 0);

// ---- purification groups --------------------------------------------------
struct alignas(8) IPair {   // a 32 x 32 tile pair (I, J), I <= J; same layout as HIP's int2
    int x, y;
};

// Per-matrix regions of the workspace.
struct MatLayout {
    double* X2;
    double* X3;
    double* T;        // native TRS4
    double* Pw;       // workspace iterate (Pb[1])
    uint8_t* planesP;
    uint8_t* planesX;
    int* expP;
    int* expX;
    uint64_t* maxP;
    uint64_t* maxX;
    uint8_t* res;     // residue products: the residues of one product, and a second
    int* expP1;       // set of exponents and row maxima of the iterates
    uint64_t* maxP1;
    double* rows;
    int* rowbad;
    double* e0;
};

constexpr int kE0Blocks = 256;   // fixed grid of the P0 / energy pass

// Everything a group of matrices (same S, kind and tile height) needs on the
// device.
struct GroupPlan {
    int count = 0;
    int S = 0;
    dmp_kind kind = DMP_OZ_INT8;
    int method = DMP_CANONICAL;
    std::vector<int> idx;             // positions in the caller's arrays
    std::vector<MatLayout> lay;
    PurDesc* pd = nullptr;            // [count]
    DevState* st = nullptr;           // [count]
    SplitDesc* splitP[2] = {nullptr, nullptr};  // [count] each
    SplitDesc* splitX = nullptr;      // [count]
    SplitDesc* splitT[2] = {nullptr, nullptr};  // TRS4: T from P (parity) and X2
    MatDesc* sq[2] = {nullptr, nullptr};
    MatDesc* up[2] = {nullptr, nullptr};
    Tile* tiles = nullptr;
    double* partials = nullptr;
    int ntiles = 0, units_rowmax = 0, units_digits = 0, max_n = 0;
    IPair* pairs = nullptr;           // 32 x 32 tile pairs I <= J of the largest matrix
    int max_pairs = 0;
    int rb = 4;                       // 32-row blocks per slice-GEMM tile (4 or 2)
    bool split_tail = true;           // the tuned table's choice for this group
    int* fix = nullptr;               // part buffer of the tail split
    int fix_pieces = 0;               // its capacity in parts
    int min_kc = 0, max_kc = 0;       // fewest / most reduction chunks of a matrix
    TailSplit tail{0, 1};             // tail split of the slice GEMMs
    int nmod = 0;                     // most moduli of its residue products (0: digit slices)
    std::vector<int> mods;            // [count] moduli of each matrix
    bool mixed = false;               // they differ
    Tile* mtiles = nullptr;           // residue GEMM tile list, nmt entries of shape mshape
    int nmt = 0, mshape = 0;
};

int native_blocks(int n);
int native_pairs(int n);
int oz_tiles(int n, int rb);

// Partition a batch into groups of equal (S, tile choice); the choice, and the
// moduli of a residue product, follow from each matrix's own (kind, S, n, nocc),
// so a matrix gets the same tiles and scales, hence bit-identical results, alone
// or in a batch.  nocc null (workspace queries, which do not know it): the same
// groups.  digits: digit slices for every matrix.
void plan_groups(int count, const int* n, const int* slices, dmp_kind kind, int method,
                 int forced_rb, std::vector<GroupPlan>& groups, const int* nocc = nullptr,
                 bool digits = false);
// Carve the workspace regions of a group (base == nullptr: measure only);
// states false: all but its device states, which the caller places.
size_t carve_group(Carver& c, GroupPlan& g, const int* n, bool states = true);

// Host copies of a group's descriptors, ready to upload.
struct GroupHost {
    std::vector<PurDesc> pd;
    std::vector<SplitDesc> sp0, sp1, sx, st0, st1;
    std::vector<MatDesc> q0, q1, u0, u1;
    std::vector<Tile> tiles, mtiles;
    std::vector<IPair> pairs;
    std::vector<uint8_t> staged;   // the bytes of the one copy to the device
};
// Fill the descriptors of a carved group for the caller's matrices; sets
// the group's tile count, unit counts, largest size and tail plan
// (``slots``: workgroups of its slice GEMM resident at once, 0 for no tail
// split).
void build_group(GroupPlan& g, const double* const* H, double* const* P, const int* n,
                 const int* nocc, int slots, GroupHost& out);

// Key of a recorded sequence of launches: every launch argument of m
// iterations of the groups follows from these values (workspace addresses
// and sizes), so equal keys mean an identical launch sequence.
std::vector<int64_t> launch_key(const std::vector<GroupPlan>& groups, int m, int device,
                                int extra);

// Iterations per replay of a recorded graph: even, so a replay ends with the
// iterate in the buffer it started from.
int iterations_per_sync(int max_n);
// The graphs (iterations of each) a run of ``predicted`` iterations launches: the
// whole multiples of m in one, then pairs.
std::vector<int> replay_plan(int m, int predicted);

// ---- caches ---------------------------------------------------------------
// Recorded graphs kept per process: those of eight launch sequences that are run
// in turn, each with its replay of m iterations, its whole multiples of m and its
// pair.
constexpr size_t kGraphsPerSequence = 3, kGraphCacheCapacity = 8 * kGraphsPerSequence;

// Thread-safe cache keyed by a vector of integers.  Holds at most
// ``capacity`` values (0: no limit); beyond that the least recently used is
// dropped.  Values are shared pointers: dropping one from the cache leaves
// it alive for a caller that still holds it, and its deleter runs when the
// last holder lets go.
template <class V>
class KeyedCache {
public:
    using Key = std::vector<int64_t>;
    using Ptr = std::shared_ptr<V>;

    explicit KeyedCache(size_t capacity = 0) : cap_(capacity) {}

    // The cached value of ``key``, or the one ``create()`` returns (stored
    // unless null).  ``create`` runs under the cache's lock, so a value is
    // created once even when threads ask for it together.
    template <class F>
    Ptr get_or_create(const Key& key, F&& create, bool* created = nullptr) {
        std::lock_guard<std::mutex> lock(mu_);
        if (created) *created = false;
        auto it = index_.find(key);
        if (it != index_.end()) {
            lru_.splice(lru_.begin(), lru_, it->second);
            return it->second->second;
        }
        Ptr v = create();
        if (!v) return v;
        if (created) *created = true;
        lru_.emplace_front(key, v);
        index_[key] = lru_.begin();
        while (cap_ > 0 && lru_.size() > cap_) {
            index_.erase(lru_.back().first);
            lru_.pop_back();
        }
        return v;
    }

    // Value of ``key`` or null; marks it as recently used.
    Ptr find(const Key& key) {
        std::lock_guard<std::mutex> lock(mu_);
        auto it = index_.find(key);
        if (it == index_.end()) return nullptr;
        lru_.splice(lru_.begin(), lru_, it->second);
        return it->second->second;
    }

    size_t size() const {
        std::lock_guard<std::mutex> lock(mu_);
        return lru_.size();
    }

    void clear() {
        std::lock_guard<std::mutex> lock(mu_);
        index_.clear();
        lru_.clear();
    }

private:
    mutable std::mutex mu_;
    size_t cap_;
    std::list<std::pair<Key, Ptr>> lru_;   // most recently used first
    std::map<Key, typename std::list<std::pair<Key, Ptr>>::iterator> index_;
};

// The one lock that serialises the purification entry points of a process
// (dmp_purify*, the batched and the taped variants and the backward pass).
std::mutex& purify_mutex();

}  // namespace dmp
