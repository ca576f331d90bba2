// Host side of the bfloat16 GEMM (gemm_bf16.h): which products it takes and
// the choice of the tile.
#include "gemm_bf16.h"

namespace clearmoe {

namespace {

// The five tiles, and what one launch of each costs on an MI355X (us), from a
// sweep of 800 products (M 100 .. 50432, N 128 .. 3072, K 160 .. 3072):
// base + full rounds * c[per_cu - 1] + the last round's c[n - 1], n being the
// workgroups of a CU in a round (at most per_cu) and c = fixed + stage * (k
// stages) + gelu.  Picking the smallest estimate costs 1.1 % over the best of
// nine tiles on that sweep, and 2.3 % without the last tile.
constexpr int kGbTiles = kTileDuo;     // those the estimate chooses from
struct GbCost {
    int bm, bn, per_cu;
    float base;
    struct {
        float fixed, stage, gelu;
    } c[3];
};
constexpr GbCost kGbCost[kGbTiles] = {
    {320, 256, 1, 0.0f, {{7.3f, 1.63f, 8.4f}}},
    {256, 256, 1, 0.0f, {{7.4f, 1.10f, 7.0f}}},
    {128, 128, 2, 2.1f, {{1.6f, 0.52f, 1.7f}, {3.2f, 0.94f, 2.4f}}},
    {64, 64, 3, 3.0f, {{0.3f, 0.27f, 0.4f}, {1.1f, 0.39f, 0.4f}, {1.5f, 0.58f, 0.5f}}},
    {128, 128, 1, 0.7f, {{3.2f, 0.48f, 1.5f}}},
};
constexpr int kGbMostRows = 320;       // of the tallest tile
constexpr int kCusPerXcd = 32;

float gb_estimate(const GbCost& t, const GemmDesc& g, int stages) {
    // a segment ends inside a tile: half a tile more for each
    const int64_t seg = g.seg_offsets != nullptr && !g.seg_merge ? g.nseg / 2 : 0;
    const int64_t mt = (g.M + t.bm - 1) / t.bm + seg, nt = (g.N + t.bn - 1) / t.bn;
    const int64_t tiles = (mt * nt + kGbXcds - 1) / kGbXcds;        // of one XCD
    const int64_t full = tiles / (kCusPerXcd * t.per_cu);
    const int64_t rest = tiles - full * kCusPerXcd * t.per_cu;
    const int64_t n = (rest + kCusPerXcd - 1) / kCusPerXcd;
    auto cost = [&](int64_t per) {
        const auto& c = t.c[per - 1];
        return c.fixed + c.stage * static_cast<float>(stages) + (g.gelu ? c.gelu : 0.0f);
    };
    return t.base + static_cast<float>(full) * cost(t.per_cu) + (n > 0 ? cost(n) : 0.0f);
}

bool gb_k_split(const GemmDesc& g) { return g.k_split < g.K || g.k_split2 < g.K; }

int gb_stages(const GemmDesc& g) {
    constexpr int BK = kGbRow / 2;
    if (!gb_k_split(g)) return (g.K + BK - 1) / BK;
    const int k1 = g.k_split < g.K ? g.k_split : g.K, k2 = g.k_split2 < g.K ? g.k_split2 : g.K;
    return (k1 + BK - 1) / BK + (k2 - k1 + BK - 1) / BK + (g.K - k2 + BK - 1) / BK;
}

// fc1 + GELU with kGbDuoTiles tiles of 256 x 128 or more (three for each of the
// 256 CUs, which hold two at a time): k_gemm_bf16_duo.  Measured against the
// best of the tiles above, N = 768 .. 3072, K = N / 4: 0.96 of its time at
// 900 tiles, 0.93 at 1200, 0.83 to 0.93 at 1200 to 4700, but 1.01 to 1.08
// at 480 to 600 tiles (one full round and a small rest).
constexpr int64_t kGbDuoTiles = 768;
int64_t gb_gelu_tiles(const GemmDesc& g) { return ((g.M + 255) / 256) * ((g.N + 127) / 128); }

template <int EPI, bool KS3>
hipError_t gb_launch(const GemmDesc& g, hipStream_t st) {
    switch (gemm_bf16_tile(g)) {
        case kTile320: return gemm_bf16_cfg<2, 4, 5, 2, 2, 2, EPI, KS3>(g, st);
        case kTile256Long:
            if constexpr (!KS3) return gemm_bf16_long<EPI>(g, st);
            return hipErrorInvalidValue;
        case kTile128: return gemm_bf16_cfg<2, 4, 2, 1, 2, 4, EPI, KS3>(g, st);
        case kTile64: return gemm_bf16_cfg<2, 2, 1, 1, 3, 3, EPI, KS3>(g, st);
        default: return gemm_bf16_cfg<2, 4, 2, 1, 3, 2, EPI, KS3>(g, st);
    }
}

// Rows of `ld` elements whose byte offsets fit a buffer descriptor.
bool fits(int64_t rows, int64_t ld) { return rows * ld * 2 < (int64_t{1} << 31); }

}  // namespace

// Everything the layer asks for in bfloat16 but operands of 2 GiB and more
// (32-bit offsets in the loads): rows of whole 16-byte pieces, parts of B at
// multiples of 8, split along n or along k, and a scale or a bias or a GELU
// (split along k only a bias, and one row stride for parts 1 and 2).
bool gemm_bf16_supported(const GemmDesc& g) {
    const bool part1 = g.n_split < g.N || g.k_split < g.K, part2 = g.n_split2 < g.N || g.k_split2 < g.K;
    if (g.K < 1 || g.N < 1 || g.M < 1 || g.M >= (int64_t{1} << 31)) return false;
    if (g.K % 8 != 0 || g.N % 8 != 0 || g.lda % 8 != 0 || g.ldc % 8 != 0) return false;
    if (g.n_split < 0 || g.n_split2 < g.n_split || g.k_split < 0 || g.k_split2 < g.k_split) return false;
    if (g.n_split % 8 != 0 || g.n_split2 % 8 != 0 || g.k_split % 8 != 0 || g.k_split2 % 8 != 0) return false;
    if (gb_k_split(g)) {
        if (g.n_split < g.N || g.n_split2 < g.N) return false;
        if (g.gelu || g.row_scale != nullptr) return false;
        if (part2 && g.ldb2 != g.ldb1) return false;
    }
    // k of each part: its rows hold as many elements (a load's scalar offset,
    // the stage's k, then lies inside the descriptor of one column's row)
    const int k1 = g.k_split < g.K ? g.k_split : g.K, k2 = g.k_split2 < g.K ? g.k_split2 : g.K;
    const int kb1 = gb_k_split(g) ? k2 - k1 : g.K, kb2 = gb_k_split(g) ? g.K - k2 : g.K;
    if (g.lda < g.K) return false;
    // a descriptor holds the rows of one tile, with a gather all of A
    const int64_t rows = g.a_rows != nullptr ? g.a_nrows : (g.M < kGbMostRows ? g.M : kGbMostRows);
    if (rows < 1 || !fits(rows, g.lda)) return false;
    if (g.n_split > 0 && g.k_split > 0 &&
        (g.B == nullptr || g.ldb % 8 != 0 || g.ldb < k1 || !fits(g.N, g.ldb)))
        return false;
    if (part1 && (g.B1 == nullptr || g.ldb1 % 8 != 0 || g.ldb1 < kb1 || !fits(g.N, g.ldb1))) return false;
    if (part2 && (g.B2 == nullptr || g.ldb2 % 8 != 0 || g.ldb2 < kb2 || !fits(g.N, g.ldb2))) return false;
    if (g.row_scale != nullptr && (g.bias != nullptr || g.gelu || g.scale_col0 % 8 != 0 || g.scale_col1 % 8 != 0))
        return false;
    if (g.c_f32 && (g.gelu || g.row_scale != nullptr)) return false;
    if (g.res != nullptr && (g.c_f32 || g.gelu || g.row_scale != nullptr || g.ldr % 8 != 0)) return false;
    return g.seg_offsets == nullptr || g.seg_merge || g.nseg <= 64;
}

GemmBf16Tile gemm_bf16_tile(const GemmDesc& g) {
    if (g.gelu && gb_gelu_tiles(g) >= kGbDuoTiles) return kTileDuo;
    const int stages = gb_stages(g);
    int best = -1;
    float t = 0.0f;
    for (int i = 0; i < kGbTiles; ++i) {
        if (gb_k_split(g) && i == kTile256Long) continue;
        const float e = gb_estimate(kGbCost[i], g, stages);
        if (best < 0 || e < t) {
            best = i;
            t = e;
        }
    }
    return static_cast<GemmBf16Tile>(best);
}

hipError_t launch_gemm_bf16(const GemmDesc& g, hipStream_t st) {
    if (gb_k_split(g)) return gb_launch<kEpiPlain, true>(g, st);
    if (g.gelu) return gemm_bf16_tile(g) == kTileDuo ? gemm_bf16_duo(g, st) : gb_launch<kEpiGelu, false>(g, st);
    if (g.row_scale != nullptr) return gb_launch<kEpiScale, false>(g, st);
    return gb_launch<kEpiPlain, false>(g, st);
}

}  // namespace clearmoe
