// Checks of the bfloat16 GEMM's host-side and address rules on the CPU, run by
// test_gemm_bf16_host.py.  Prints each violation; exits with 1 if any.
#include <cstdio>
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

int main(int argc, char** argv) {
    if (argc > 1 && std::strcmp(argv[1], "parts") == 0) parts();
    else return 2;
    std::printf("%d violations\n", g_bad);
    return g_bad != 0;
}
