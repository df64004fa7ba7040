// What the host and the kernels of the biased schemes have to agree on: how a
// line is cut into lane partitions, which instance of the wave kernel runs it,
// and how many elements of LDS a wave of that instance touches.
#pragma once

#include <algorithm>
#include <vector>

#include "cfd_internal.h"

#ifdef __HIPCC__
#define CFD_HOST_DEVICE __host__ __device__
#else
#define CFD_HOST_DEVICE
#endif

namespace cfd {

// x lines of a wave are moved in at most this many passes of 64 lanes.
constexpr int kRowPass = 16;
// Rows of a lane's partition, at most, and log2 of a line's partitions.
constexpr int kBiasMaxL = 12, kBiasMaxLgP = 6;
static_assert((kBiasMaxL << kBiasMaxLgP) <= kBiasMaxPow, "the power tables cover the wave kernel's lines");

// The fewest partitions of at most 12 rows, the rows spread evenly (L or L - 1
// per partition): fewer partitions keep the stencil halo's share of the loads
// down, and 12 rows of a pair of biases are what fits a quarter of a SIMD's
// registers.  y and z lines stop at 16 partitions: with fewer than 4 lines per
// wave their accesses cover less than 32 contiguous bytes, and the sweep
// kernel, 64 lines per wave, takes over (not with an embedded second
// derivative, which only the wave kernel solves; those lines end at 256 nodes).
// x lines take more where that keeps a wave's rows, ghosts included, at
// kRowPass passes or fewer.  False: the sweep kernel takes the lines.
inline bool bias_split(int N, int dir, int emb, BiasSplit &s) {
    if (N < 2) return false;
    for (int lg = 0; lg <= (dir == 0 || emb ? kBiasMaxLgP : 4); ++lg) {
        const int L = (N + (1 << lg) - 1) >> lg;
        if (L > kBiasMaxL) continue;
        if (dir == 0) {
            const int Tn = N + 2 * (kBiasHalf + 1);   // at most
            const int rows = 64 >> lg, per = Tn > 32 ? 1 : Tn > 16 ? 2 : 4;
            if ((rows + per - 1) / per * ((Tn + 63) / 64) > kRowPass) continue;
            if (L < 2) return false;
        }
        s.lgP = lg;
        s.L = L;
        return true;
    }
    return false;
}

// Half-width of the kernel instance that runs a launch: the launch's own class,
// whatever the offsets' width.  An instance of a wider class would stage more
// ghosts than the class needs and multiply them by zero weights.
inline int bias_instance_half(const BiasLaunch &g) { return g.hb; }

// Ghosts either side that an instance of half-width hb stages with an x line
// (closure rows reach one node further than the interior).
CFD_HOST_DEVICE inline int bias_ghosts(int ng, int hb, int periodic) { return periodic ? 0 : ng < hb + 1 ? ng : hb + 1; }

// Elements of one wave's LDS tile (x lines; 0 along y and z) for an instance of
// half-width hb: its lines' columns at an odd pitch; a partition short of a row
// reads one element past it.
inline int bias_tile_elems(const BiasSplit &s, int dir, int hb, int ng, int periodic, int N) {
    if (dir != 0) return 0;
    return (64 >> s.lgP) * ((N + 2 * bias_ghosts(ng, hb, periodic)) | 1) + 2;
}

// A run of fields [f0, f1) of one block, or one field's part-th of parts runs
// of lines (every operator's lines cut alike), and its cost.
struct BiasUnit {
    int block, f0, f1, part, parts;
    int64_t cost;
    int queue;
};

// Deals the work of one launch to XCD queues; cost[b][f]: its nodes of field f
// of block b.  A unit of several fields is at most 1/32 of a queue's share; its
// block-fields' lines of every direction then share one L2, and the velocity
// comes from the last-level cache (64 blocks, 22 fields, X_2 pair, FP64: 454 us;
// units of a third of a share 463).  Units go to the least loaded queue, largest
// first.  Where that leaves a queue above 1.3 times the mean (few block-fields,
// or few large ones, for the queues), block-fields are cut into runs of lines of
// at most 1/8 of a share: whole ones left dies idle (one field of 128^3, one
// bias, FP64: 136 us on one die, 22 cut; three fields of 64^3 with the X_2 pair
// 24.5 and 11.8; six of 128 x 96 x 80 88 and 64).  Runs of 1/4 of a share take 86 us
// where these take 77 (three fields of 128^3, pair), runs of 1/32 17.7 where these
// take 11.7 (one field of 96^3, pair).
inline std::vector<BiasUnit> bias_deal(const std::vector<std::vector<int64_t>> &cost, int queues) {
    int64_t total = 0;
    for (const auto &b : cost)
        for (int64_t c : b) total += c;
    std::vector<BiasUnit> units;
    auto deal = [&](int64_t most) {   // fields of more than most nodes in parts
        units.clear();
        for (int b = 0; b < (int)cost.size(); ++b) {
            BiasUnit u{b, 0, 0, 0, 1, 0, 0};
            auto flush = [&](int f) {
                if (u.cost > 0) units.push_back(u);
                u = BiasUnit{b, f, f, 0, 1, 0, 0};
            };
            for (int f = 0; f < (int)cost[b].size(); ++f) {
                const int64_t c = cost[b][f];
                if (u.cost > 0 && u.cost + c > total / (32 * queues)) flush(f);
                if (c > most) {
                    flush(f);
                    const int parts = (int)((c + most - 1) / most);
                    for (int k = 0; k < parts; ++k) units.push_back(BiasUnit{b, f, f + 1, k, parts, c / parts, 0});
                    u.f0 = u.f1 = f + 1;
                    continue;
                }
                u.cost += c;
                u.f1 = f + 1;
            }
            flush(0);
        }
        std::vector<size_t> ord(units.size());
        for (size_t i = 0; i < ord.size(); ++i) ord[i] = i;
        std::stable_sort(ord.begin(), ord.end(), [&](size_t x, size_t y) { return units[x].cost > units[y].cost; });
        std::vector<int64_t> load(queues, 0);
        for (size_t i : ord) {
            units[i].queue = (int)(std::min_element(load.begin(), load.end()) - load.begin());
            load[units[i].queue] += units[i].cost;
        }
        return *std::max_element(load.begin(), load.end());
    };
    if (total == 0) return units;
    if (10 * queues * deal(total) > 13 * total) deal(std::max<int64_t>(1, total / (8 * queues)));
    return units;
}

}  // namespace cfd
