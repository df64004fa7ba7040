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

// Work dealt to the queues: every line of every field once, no queue above 1.3 times the mean.
static void queues() {
    unsigned rng = 12345;
    auto next = [&](int n) { return (int)((rng = rng * 1664525u + 1013904223u) >> 8) % n; };
    for (int rep = 0; rep < 3000; ++rep) {
        const int nb = 1 + (rep % 3 == 0 ? 0 : next(12)), nf = 1 + next(rep % 2 ? 3 : 24);
        std::vector<std::vector<int64_t>> cost(nb, std::vector<int64_t>(nf));
        int64_t total = 0;
        for (auto &b : cost) {
            const int64_t n = 4096 + next(2000000);
            for (int64_t &c : b) total += c = n * next(4);   // operators that select some fields only
        }
        const std::vector<BiasUnit> units = bias_deal(cost, 8);
        std::vector<int64_t> load(8, 0);
        std::vector<std::vector<double>> seen(nb, std::vector<double>(nf, 0.0));
        for (const BiasUnit &u : units) {
            EXPECT(u.queue >= 0 && u.queue < 8 && u.f0 < u.f1 && u.part >= 0 && u.part < u.parts);
            EXPECT(u.parts == 1 || u.f1 == u.f0 + 1);
            load[u.queue] += u.cost;
            for (int f = u.f0; f < u.f1; ++f) seen[u.block][f] += 1.0 / u.parts;
        }
        for (int b = 0; b < nb; ++b)
            for (int f = 0; f < nf; ++f)
                EXPECT(cost[b][f] == 0 || (seen[b][f] > 0.999 && seen[b][f] < 1.001));
        for (int64_t l : load) EXPECT(10 * 8 * l <= 13 * total);
    }
}

int main() {
    tiles();
    queues();
    std::printf("%s (%d failures)\n", g_fail ? "FAIL" : "OK", g_fail);
    return g_fail ? 1 : 0;
}
