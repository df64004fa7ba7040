// What the host and the kernels of the biased schemes have to agree on: how a
// line is cut into lane partitions, which instance of the wave kernel runs it,
// and how many elements of LDS a wave of that instance touches.
#pragma once

#include <algorithm>

#include "cfd_internal.h"

#ifdef __HIPCC__
#define CFD_HOST_DEVICE __host__ __device__
#else
#define CFD_HOST_DEVICE
#endif

namespace cfd {

// x lines of a wave are moved in at most this many passes of 64 lanes.
constexpr int kRowPass = 16;

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
    for (int lg = 0; lg <= (dir == 0 || emb ? 6 : 4); ++lg) {
        const int L = (N + (1 << lg) - 1) >> lg;
        if (L > 12) continue;
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

}  // namespace cfd
