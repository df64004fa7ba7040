// Host-side rules of the biased schemes (csrc/cfd_biased_plan.h), without a GPU.
#include <cstdio>
#include <vector>

#include "cfd_biased_plan.h"

using namespace cfd;

static int g_fail = 0;
#define EXPECT(c)                                                                \
    do {                                                                         \
        if (!(c)) {                                                              \
            if (++g_fail < 20) std::printf("FAIL %s:%d %s\n", __FILE__, __LINE__, #c); \
        }                                                                        \
    } while (0)

// Every index of its LDS tile that a wave of the kernel uses on x lines, against the tile the host allots.
static void tiles() {
    for (int big = 0; big <= 1; ++big)
        for (int emb = 0; emb <= 1; ++emb)
            for (int hb = emb ? 3 : 2; hb <= 5; ++hb)
                for (int periodic = 0; periodic <= 1; ++periodic)
                    for (int ng = periodic ? 0 : hb; ng <= (periodic ? 0 : 9); ++ng)
                        for (int N = 2; N <= 800; ++N) {
                            BiasSplit sp;
                            if (!bias_split(N, 0, emb, sp)) {
                                EXPECT(N > 768);
                                continue;
                            }
                            BiasLaunch g;
                            g.hb = hb;
                            g.emb = emb;
                            g.big = big;
                            const int HB = bias_instance_half(g);
                            EXPECT(HB == hb);   // a wider instance would read ghosts that the scheme does not
                            const int tilew = bias_tile_elems(sp, 0, HB, ng, periodic, N);
                            const int P = 1 << sp.lgP, NW = 64 >> sp.lgP, L = sp.L;
                            const int nfull = N - P * (L - 1);
                            EXPECT(nfull >= 1 && nfull <= P && L >= 2 && L <= 12);
                            const int e = bias_ghosts(ng, HB, periodic), Tn = N + 2 * e, tp = Tn | 1;
                            int most = (NW - 1) * tp + Tn - 1;   // rows staged
                            const bool lastfull = nfull == P;
                            for (int p = 0; p < P; ++p) {
                                const int k0 = p * (L - 1) + std::min(p, nfull), base = (NW - 1) * tp;
                                if (!periodic) {
                                    const bool whole = e > HB || (e == HB && lastfull);
                                    for (int t = 0; t < L + 2 * HB; ++t) {
                                        const int j = k0 - HB + t;
                                        if (!whole && !(j >= -e && j < N + e)) continue;
                                        EXPECT(j + e >= 0 && j + e < Tn);
                                        most = std::max(most, base + j + e);
                                    }
                                }
                                most = std::max(most, (NW - 1) * (N | 1) + k0 + L - 1);   // velocity rows read, one past
                            }
                            EXPECT(most < tilew);
                        }
}

int main() {
    tiles();
    std::printf("%s (%d failures)\n", g_fail ? "FAIL" : "OK", g_fail);
    return g_fail ? 1 : 0;
}
