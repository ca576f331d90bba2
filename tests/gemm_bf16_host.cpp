// Checks of the bfloat16 GEMM's host-side and address rules on the CPU, run by
// test_gemm_bf16_host.py.  Prints each violation; exits with 1 if any.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "kernels.h"

using namespace clearmoe;

static int g_bad = 0;
static void expect(bool ok, const char* what, int a, int b, int c, int d) {
    if (!ok && ++g_bad <= 20) std::printf("%s: %d %d %d %d\n", what, a, b, c, d);
}

// Every load of B goes through a buffer descriptor that holds the load's
// scalar offset (the k of its stage) whatever the columns: also the columns
// past N of a short last tile, whose lanes ask for an offset past the end.
// A range check that takes the scalar offset off the size must not wrap.
static void parts() {
    constexpr int kStage = 64;                           // k per stage
    for (int r = 0; r <= 136; r += 8)
        for (int q = 0; q <= 72; q += 8)
            for (int pair = 0; pair < 3; ++pair) {       // one part, [r | q], [r | q | q]
                const int N = pair == 0 ? r : r + pair * q;
                if (N == 0) continue;
                GemmDesc g = gemm_desc(1000, N, 1024);
                if (pair >= 1) g.n_split = r;
                if (pair == 2) g.n_split2 = r + q;
                const int cols[3] = {pair == 0 ? N : r, pair >= 1 ? q : 0, pair == 2 ? q : 0};
                for (int bn = 64; bn <= 256; bn *= 2)
                    for (int ng = 0; ng < (N + bn - 1) / bn * bn; ng += 8) {
                        const GemmBPart b = gemm_b_part(N, g.n_split, g.n_split2, ng);
                        expect(b.part >= 0 && b.part <= 2 && b.n1 - b.n0 == cols[b.part], "columns of a part",
                               r, q, pair, ng);
                        if (ng < N) {
                            const int want = ng < cols[0] ? 0 : ng < cols[0] + cols[1] ? 1 : 2;
                            expect(b.part == want && ng >= b.n0 && ng < b.n1, "part", r, q, pair, ng);
                        } else {
                            expect(ng >= b.n1, "columns past N", r, q, pair, ng);
                        }
                        const long bytes = static_cast<long>(b.n1 - b.n0) * g.K * 2;
                        const long soff = (g.K - 1) / kStage * kStage * 2L;
                        expect(soff < bytes, "scalar offset past the descriptor", r, q, pair, ng);
                    }
            }
}

// A [r | q | q] product split along k, as the pair order's y product.
static GemmDesc k_split_desc() {
    static unsigned char mem[16];
    GemmDesc g = gemm_desc(1000, 384, 128 + 2 * 32);
    g.A = mem; g.lda = g.K;
    g.B = mem; g.ldb = 128;
    g.B1 = mem; g.ldb1 = 32;
    g.B2 = mem; g.ldb2 = 32;
    g.k_split = 128;
    g.k_split2 = 128 + 32;
    g.C = mem; g.ldc = g.N;
    return g;
}

// What the bfloat16 kernels say they take, their launch takes and they compute.
static void supported() {
    const GemmDesc y = k_split_desc();
    expect(gemm_bf16_supported(y), "a k split", 0, 0, 0, 0);
    GemmDesc g = y;
    g.gelu = 1;
    expect(!gemm_bf16_supported(g), "a k split with a GELU", 0, 0, 0, 0);
    g = y;
    g.row_scale = reinterpret_cast<const float*>(g.A);
    g.scale_rows = reinterpret_cast<const int32_t*>(g.A);
    expect(!gemm_bf16_supported(g), "a k split with a scale", 0, 0, 0, 0);
    g = y;
    g.ldb2 = 40;                                         // the kernel has one row stride for parts 1 and 2
    expect(!gemm_bf16_supported(g), "a k split with two row strides", 0, 0, 0, 0);
    g = y;
    g.k_split2 = g.K;                                    // [r | 2q]: one part less, its stride free
    g.ldb1 = 64;
    g.ldb2 = 0;
    g.B2 = nullptr;
    expect(gemm_bf16_supported(g), "a k split in two", 0, 0, 0, 0);
    // rows shorter than the part: a load's scalar offset would leave the
    // descriptor of a part of few columns
    g = y;
    g.ldb = 120;
    expect(!gemm_bf16_supported(g), "short rows of B", 0, 0, 0, 0);
    g = y;
    g.ldb1 = g.ldb2 = 24;
    expect(!gemm_bf16_supported(g), "short rows of B1 and B2", 0, 0, 0, 0);
    g = y;
    g.lda = g.K - 8;
    expect(!gemm_bf16_supported(g), "short rows of A", 0, 0, 0, 0);
}

// Few rows far apart (class tokens of a long sequence: the class rows of z, H
// times the stride apart) stay with the bfloat16 kernels as long as the rows of
// one tile lie within 2 GiB.
static void far_rows() {
    static unsigned char mem[16];
    for (int m : {1, 13, 320, 5000}) {
        GemmDesc g = gemm_desc(m, 768, 3072);
        g.A = mem;
        g.B = mem; g.ldb = g.K;
        g.C = mem; g.ldc = g.N;
        const int64_t rows = m < 320 ? m : 320;          // of the tallest tile
        const int64_t most = (int64_t{1} << 30) / rows;  // elements apart
        g.lda = (most - 1) / 8 * 8;
        expect(gemm_bf16_supported(g), "rows within 2 GiB", m, static_cast<int>(g.lda), 0, 0);
        g.lda = (most + 7) / 8 * 8;
        expect(!gemm_bf16_supported(g), "rows past 2 GiB", m, static_cast<int>(g.lda), 0, 0);
    }
}

// The tile of each product in argv: M N K gelu nseg k_split k_split2 (nseg 0:
// not grouped).
static int tiles(int n, char** v) {
    static const char* names[] = {"320", "256 long", "128", "64", "128 deep", "duo"};
    static int32_t seg[1];
    for (int i = 0; i + 6 < n; i += 7) {
        GemmDesc g = gemm_desc(std::atoll(v[i]), std::atoi(v[i + 1]), std::atoi(v[i + 2]));
        g.gelu = std::atoi(v[i + 3]);
        g.nseg = std::atoi(v[i + 4]);
        g.seg_offsets = g.nseg > 0 ? seg : nullptr;
        g.k_split = std::atoi(v[i + 5]);
        g.k_split2 = std::atoi(v[i + 6]);
        std::printf("%s\n", names[gemm_bf16_tile(g)]);
    }
    return 0;
}

int main(int argc, char** argv) {
    if (argc > 1 && std::strcmp(argv[1], "tiles") == 0) return tiles(argc - 2, argv + 2);
    if (argc > 1 && std::strcmp(argv[1], "parts") == 0) parts();
    else if (argc > 1 && std::strcmp(argv[1], "supported") == 0) supported();
    else if (argc > 1 && std::strcmp(argv[1], "far_rows") == 0) far_rows();
    else return 2;
    std::printf("%d violations\n", g_bad);
    return g_bad != 0;
}
