// C-ABI entry points of the Ozaki-scheme GEMM (Sec. 2.4).
#include <algorithm>
#include <cstring>
#include <vector>

#include "host.hpp"

namespace dmp {

namespace {

struct GemmLayout {
    uint8_t* pa;
    uint8_t* pb;
    int* ea;
    int* eb;
    uint64_t* ma;
    uint64_t* mb;
    int* fix;          // part buffer of the split tail (nullable)
    TailSplit tail;
};

// Split tail of the m x n product's tiles on the current device; the
// workspace query and the launch take the same plan, so the part buffer is
// only as large as the launch needs (none when the tiles fill whole rounds).
TailSplit gemm_tail(int m, int n, int k, int s, dmp_kind kind) {
    const int rb = gemm_tile_blocks(m, n, s, kind);
    const int tiles = m > 0 && n > 0 ? tile_rows(m, 32 * rb) * tile_cols(n) : 0;
    TailSplit t{tiles, 1};
    if ((kind != DMP_OZ_INT8 && kind != DMP_OZ_FP16) || k <= 0 || tiles == 0 ||
        !tail_split_enabled())
        return t;
    const int kc = int(chunks_of(k, kind));
    const int cap = tail_split_capacity(tiles, kc, rb);
    int slots = 0;
    if (cap <= 0 || resident_slots(s, kind, rb, &slots) != DMP_OK) {
        clear_error();
        return t;
    }
    return plan_gemm_split(tiles, slots, kc, cap);
}

// ``split``: plan a split tail (single products; the grouped launch keeps
// its tiles whole)
GemmLayout carve_gemm(Carver& c, int m, int n, int k, int s, dmp_kind kind, bool split = false) {
    GemmLayout g;
    g.tail = split ? gemm_tail(m, n, k, s, kind) : TailSplit{0, 1};
    g.pa = c.take<uint8_t>(plane_bytes(m, k, s, kind));
    g.pb = c.take<uint8_t>(plane_bytes(n, k, s, kind));
    g.ea = c.take<int>(round_up(m, kPad));
    g.eb = c.take<int>(round_up(n, kPad));
    g.ma = c.take<uint64_t>(round_up(m, kPad));
    g.mb = c.take<uint64_t>(round_up(n, kPad));
    const int rb = gemm_tile_blocks(m, n, s, kind);
    const int tiles = m > 0 && n > 0 ? tile_rows(m, 32 * rb) * tile_cols(n) : 0;
    const size_t parts = g.tail.nsplit > 1 ? size_t(tiles - g.tail.nfull) * g.tail.nsplit : 0;
    g.fix = parts > 0 ? c.take<int>(parts * piece_ints(s, rb)) : nullptr;
    return g;
}

__global__ void k_zero_rows(double* c, int m, int n, int ldc) {
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < int64_t(m) * n) c[(i / n) * ldc + i % n] = 0.0;
}

bool is_trans(char t) { return t == 'T' || t == 't'; }
bool valid_trans(char t) { return t == 'N' || t == 'n' || t == 'T' || t == 't'; }

}  // namespace

}  // namespace dmp

using namespace dmp;

extern "C" {

size_t dmp_gemm_workspace_bytes(int m, int n, int k, int slices, dmp_kind kind) {
    if (kind == DMP_FP64_NATIVE) return 256;
    if (m < 0 || n < 0 || k < 0 || slices < 1 || slices > kMaxSlices) return 0;
    if (kind == DMP_MARKIDIS_FP16 && slices > kMaxTerms) return 0;
    Carver c(nullptr);
    carve_gemm(c, m, n, k, slices, kind, true);
    return c.used();
}

int dmp_ozaki_gemm(char transA, char transB, int m, int n, int k, const double* A, int lda,
                   const double* B, int ldb, double* C, int ldc, int slices, dmp_kind kind,
                   void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    hipStream_t s = static_cast<hipStream_t>(stream);
    DMP_CHECK(check_kind_slices(kind, slices));
    if (!valid_trans(transA) || !valid_trans(transB)) {
        set_error("trans must be 'N' or 'T'");
        return DMP_EINVAL;
    }
    if (m < 0 || n < 0 || k < 0) {
        set_error("negative size");
        return DMP_EINVAL;
    }
    const bool ta = is_trans(transA), tb = is_trans(transB);
    const int a_cols = ta ? m : k, b_cols = tb ? k : n;
    if (lda < std::max(1, a_cols) || ldb < std::max(1, b_cols) || ldc < std::max(1, n)) {
        set_error("leading dimension too small");
        return DMP_EINVAL;
    }
    if (m == 0 || n == 0) return DMP_OK;
    if (C == nullptr || (k > 0 && (A == nullptr || B == nullptr))) {
        set_error("null matrix pointer");
        return DMP_EINVAL;
    }
    if (k == 0) {
        const int64_t tot = int64_t(m) * n;
        k_zero_rows<<<unsigned((tot + 255) / 256), 256, 0, s>>>(C, m, n, ldc);
        DMP_CHECK_HIP(hipGetLastError());
        return DMP_OK;
    }
    if (kind == DMP_FP64_NATIVE) return native_dgemm(s, ta, tb, m, n, k, A, lda, B, ldb, C, ldc);
    if (k > max_k_for(slices, kind)) {
        set_error("k = %d exceeds the exact INT32 range for %d slices (max %lld)", k, slices,
                  (long long)max_k_for(slices, kind));
        return DMP_EINVAL;
    }
    if (m > 65535 * kTileN || n > 65535 * kTileN) {
        set_error("matrix too large");
        return DMP_EINVAL;
    }
    const size_t need = dmp_gemm_workspace_bytes(m, n, k, slices, kind);
    if (ws == nullptr || ws_bytes < need) {
        set_error("workspace of %zu bytes required", need);
        return DMP_ENOMEM;
    }
    DMP_CHECK(check_workspace_alignment(ws));
    Carver c(ws);
    GemmLayout g = carve_gemm(c, m, n, k, slices, kind, true);
    const int KC = int(chunks_of(k, kind));
    const int64_t rb_stride = int64_t(KC) * planes_of(slices, kind) * kFragBytes;

    SplitDesc da{};
    da.A = A;
    da.lda = lda;
    da.R = m;
    da.K = k;
    da.trans = ta ? 1 : 0;
    da.KC = KC;
    da.maxbits = g.ma;
    da.expo = g.ea;
    da.planes = g.pa;
    da.state_index = -1;
    SplitDesc db = da;
    db.A = B;
    db.lda = ldb;
    db.R = n;
    db.trans = tb ? 0 : 1;   // operand row j = column j of op(B)
    db.maxbits = g.mb;
    db.expo = g.eb;
    db.planes = g.pb;
    DMP_CHECK(launch_split_pair(da, db, slices, kind, s));

    // the tile of a block follows from its number: no tile list
    const int rb = gemm_tile_blocks(m, n, slices, kind);
    const int tm = tile_rows(m, 32 * rb), tn = tile_cols(n);
    GemmParams p{};
    p.tm = tm;
    p.tn = tn;
    p.descs = nullptr;
    p.one.pa = g.pa;
    p.one.pb = g.pb;
    p.one.ea = g.ea;
    p.one.eb = g.eb;
    p.one.out = C;
    p.one.a_rb_stride = rb_stride;
    p.one.b_rb_stride = rb_stride;
    p.one.M = m;
    p.one.N = n;
    p.one.KC = KC;
    p.one.ldc = ldc;
    p.one.state_index = -1;
    p.mode = EPI_STORE;
    if (g.fix != nullptr) {
        p.fix = g.fix;
        p.nfull = g.tail.nfull;
        p.nsplit = g.tail.nsplit;
    }
    return launch_ozgemm(slices, kind, p, tm * tn, s, rb);
}

// ---------------------------------------------------------------------------
// Grouped GEMM: every phase is one launch over all products.

size_t dmp_gemm_batched_workspace_bytes(int count, const int* m, const int* n, const int* k,
                                        int slices, dmp_kind kind) {
    if (count < 0 || slices < 1 || slices > kMaxSlices) return 0;
    if (kind == DMP_MARKIDIS_FP16 && slices > kMaxTerms) return 0;
    if (count > 0 && (!m || !n || !k)) return 0;
    for (int b = 0; b < count; ++b)
        if (m[b] < 1 || n[b] < 1 || k[b] < 1) return 0;
    Carver c(nullptr);
    size_t tiles = 0;
    for (int b = 0; b < count; ++b) {
        if (kind != DMP_FP64_NATIVE) carve_gemm(c, m[b], n[b], k[b], slices, kind);
        tiles += size_t(tile_rows(m[b], 64)) * size_t(tile_cols(n[b]));   // the lower tile height
    }
    c.take<SplitDesc>(2 * size_t(count));
    c.take<MatDesc>(count);
    c.take<Tile>(std::max<size_t>(1, tiles));
    return c.used();
}

int dmp_ozaki_gemm_batched(int count, const int* m, const int* n, const int* k,
                           const double* const* A, const double* const* B, double* const* C,
                           int slices, dmp_kind kind, void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    hipStream_t s = static_cast<hipStream_t>(stream);
    DMP_CHECK(check_kind_slices(kind, slices));
    if (count < 0 || (count > 0 && (!m || !n || !k || !A || !B || !C))) {
        set_error("bad batch arguments");
        return DMP_EINVAL;
    }
    for (int b = 0; b < count; ++b) {
        if (m[b] < 1 || n[b] < 1 || k[b] < 1 || !A[b] || !B[b] || !C[b]) {
            set_error("batch entry %d: sizes must be >= 1 and pointers non-null", b);
            return DMP_EINVAL;
        }
        if (kind != DMP_FP64_NATIVE && k[b] > max_k_for(slices, kind)) {
            set_error("batch entry %d: k too large for %d slices", b, slices);
            return DMP_EINVAL;
        }
    }
    if (count == 0) return DMP_OK;
    if (kind == DMP_FP64_NATIVE) {
        for (int b = 0; b < count; ++b)
            DMP_CHECK(native_dgemm(s, false, false, m[b], n[b], k[b], A[b], k[b], B[b], n[b], C[b], n[b]));
        return DMP_OK;
    }
    const size_t need = dmp_gemm_batched_workspace_bytes(count, m, n, k, slices, kind);
    if (ws == nullptr || ws_bytes < need) {
        set_error("workspace of %zu bytes required", need);
        return DMP_ENOMEM;
    }
    DMP_CHECK(check_workspace_alignment(ws));
    Carver c(ws);
    std::vector<GemmLayout> lay(count);
    for (int b = 0; b < count; ++b) lay[b] = carve_gemm(c, m[b], n[b], k[b], slices, kind);
    // operands: all left ones, then all right ones
    std::vector<SplitDesc> sd(2 * size_t(count));
    std::vector<MatDesc> md(count);
    std::vector<Tile> tiles;
    for (int b = 0; b < count; ++b) {
        const int KC = int(chunks_of(k[b], kind));
        SplitDesc d{};
        d.A = A[b];
        d.lda = k[b];
        d.R = m[b];
        d.K = k[b];
        d.trans = 0;
        d.KC = KC;
        d.maxbits = lay[b].ma;
        d.expo = lay[b].ea;
        d.planes = lay[b].pa;
        d.state_index = -1;
        sd[b] = d;
        // B's operand rows are its columns: transpose the digit read by
        // splitting B^T, i.e. columns of the row-major k x n matrix.
        d.A = B[b];
        d.lda = n[b];
        d.R = n[b];
        d.trans = 1;
        d.maxbits = lay[b].mb;
        d.expo = lay[b].eb;
        d.planes = lay[b].pb;
        sd[count + b] = d;
        MatDesc q{};
        q.pa = lay[b].pa;
        q.pb = lay[b].pb;
        q.ea = lay[b].ea;
        q.eb = lay[b].eb;
        q.out = C[b];
        q.a_rb_stride = int64_t(KC) * planes_of(slices, kind) * kFragBytes;
        q.b_rb_stride = q.a_rb_stride;
        q.M = m[b];
        q.N = n[b];
        q.KC = KC;
        q.ldc = n[b];
        q.state_index = -1;
        md[b] = q;
    }
    SplitUnits units;
    count_split_units(sd.data(), int(sd.size()), units);
    const bool self = split_takes_maxima(sd.data(), int(sd.size()));
    if (self)
        for (SplitDesc& d : sd) d.maxbits = nullptr;
    // tiles of the longest reductions first (dispatched in that order)
    const int rb = batch_tile_blocks(count, m, n, slices, kind);
    std::vector<int> order(count);
    for (int b = 0; b < count; ++b) order[b] = b;
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return k[x] > k[y]; });
    for (int b : order)
        append_tiles(tiles, tile_rows(m[b], 32 * rb), tile_cols(n[b]), false, uint32_t(b), 32 * rb);
    // descriptors and tiles in one copy
    SplitDesc* sd_dev = c.take<SplitDesc>(2 * size_t(count));
    MatDesc* md_dev = c.take<MatDesc>(count);
    Tile* t_dev = c.take<Tile>(tiles.size());
    const uint8_t* base = reinterpret_cast<const uint8_t*>(sd_dev);
    std::vector<uint8_t> staged(size_t(reinterpret_cast<const uint8_t*>(t_dev) - base) + tiles.size() * sizeof(Tile));
    std::memcpy(staged.data(), sd.data(), sd.size() * sizeof(SplitDesc));
    std::memcpy(staged.data() + (reinterpret_cast<const uint8_t*>(md_dev) - base), md.data(), md.size() * sizeof(MatDesc));
    std::memcpy(staged.data() + (reinterpret_cast<const uint8_t*>(t_dev) - base), tiles.data(),
                tiles.size() * sizeof(Tile));
    // the host copy must outlive the asynchronous one (the stream is drained
    // before any error return); the launches below stay asynchronous
    const hipError_t e = hipMemcpyAsync(sd_dev, staged.data(), staged.size(), hipMemcpyHostToDevice, s);
    const hipError_t e_sync = hipStreamSynchronize(s);
    DMP_CHECK_HIP(e);
    DMP_CHECK_HIP(e_sync);
    DMP_CHECK(launch_split_set(sd_dev, 2 * count, units, !self, slices, kind, s));
    GemmParams p{};
    p.tiles = t_dev;
    p.descs = md_dev;
    p.mode = EPI_STORE;
    p.spread = count > 1 ? 1 : 0;
    DMP_CHECK(launch_ozgemm(slices, kind, p, int(tiles.size()), s, rb));
    return DMP_OK;
}

}  // extern "C"
