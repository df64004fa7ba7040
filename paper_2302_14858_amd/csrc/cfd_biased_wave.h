// Wave kernel of the biased schemes (cfd_biased.hip states the systems): a
// wave owns 64 / P lines of one field, P = 1 .. 64 a power of two, and its
// lanes are the P partitions of those lines (lane = partition * (64 / P) +
// line, 2 to 12 rows each).  A lane issues every load of its rows
// and their stencil halo before any arithmetic and keeps them in registers.
// Each bias is solved locally with a zero value entering the partition (the
// closure rows where the lane holds them); the exact solution is the local one
// plus (-alpha)^distance times the true value entering it, which a scan over
// the partitions' local end values with the constant weight (-alpha)^rows
// gives by lane shuffles (around the line on periodic lines, closed by
// 1 / (1 - (-alpha)^N)).  Consecutive lines of y and z are consecutive x, so
// their accesses run along the contiguous direction; x lines are staged
// through a piece of LDS that only this wave uses, filled and drained with
// contiguous accesses.  So a wave never waits for another: there is no
// workgroup barrier, and the phases of one wave (loads, solve, stores) overlap
// the others'.  One launch takes every direction and length of a plan's
// operators with one stencil class.
//
// W schemes solve their embedded second derivative in the same registers: its
// constant-coefficient tridiagonal system splits into a forward and a backward
// bidiagonal recurrence of the same form.
#pragma once

#include <climits>

#include <hip/hip_runtime.h>

#include "cfd_biased_plan.h"

namespace cfd {
namespace {

// Orders the LDS accesses of one wave (its LDS operations execute in order, so
// only the compiler has to keep them so); no other wave shares the tile.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The same address, unknown to the compiler: what is read through it is not
// loaded earlier, so wave-uniform values of the last phase do not hold scalar
// registers (or, out of those, vector lanes) through the first; and the steps
// of a walking base stay in scalar registers beside a lane's fixed offset.
template <typename P>
__device__ __forceinline__ P *later(P *p) {
    asm volatile("" : "+s"(p));
    return p;
}
// Plan tables, which no kernel writes, in the constant address space: their
// wave-uniform values are read by scalar loads also after a store.
#define CONST_AS __attribute__((address_space(4)))
template <typename P>
__device__ __forceinline__ const CONST_AS P *later(const CONST_AS P *p) {
    uint64_t a = (uint64_t)p;
    asm volatile("" : "+s"(a));
    return (const CONST_AS P *)a;
}

// The x lines of a wave are moved row by row: a pass of the wave covers 64
// columns of one row, or two or four rows of at most 32 or 16, and its addresses
// take a wave-uniform step (walking the rows' elements 64 at a time took 95
// vector instructions per output row, twice the solve).  bias_split keeps the
// passes at kRowPass or fewer.
struct RowMap {
    int cols, nval, lgr;   // columns, real rows, log2 of rows per pass
    int sub, col;          // this lane's row in a pass and column
    int npass;
    bool whole;            // one pass per row or more, every row real
    __device__ __forceinline__ RowMap(int cols_, int nval_, int NW, int lane) : cols(cols_), nval(nval_) {
        lgr = cols > 32 ? 0 : cols > 16 ? 1 : 2;
        sub = lane >> (6 - lgr);
        col = lane & ((64 >> lgr) - 1);
        npass = (NW >> lgr) * ((cols + 63) >> 6);
        whole = cols <= 64 && nval == NW && (npass & 3) == 0;
    }
    // Whole maps: fn(i, at): in pass i this lane's element lies at from its first
    // one's, step from row to row.
    template <typename U, typename Fn>
    __device__ __forceinline__ void each(U step, Fn fn) const {
        if (col < cols) {
            U at = 0;
#pragma unroll
            for (int i0 = 0; i0 < kRowPass; i0 += 4)
                if (i0 < npass) {
#pragma unroll
                    for (int i = i0; i < i0 + 4; ++i) {
                        fn(i, at);
                        at += step << lgr;
                    }
                }
        }
    }
    // Any map: fn(i, row, column) for the elements that exist.
    template <typename Fn>
    __device__ __forceinline__ void any(Fn fn) const {
        int r = 0, c = 0;
#pragma unroll
        for (int i = 0; i < kRowPass; ++i)
            if (i < npass) {
                if (c + col < cols && r + sub < nval) fn(i, r + sub, c + col);
                const bool last = c + 64 >= cols;
                r += last ? 1 << lgr : 0;
                c = last ? 0 : c + 64;
            }
    }
};
// Rows from src (the first line's column 0; the first line is row u0 of its
// plane) into val, all requested before any is used (elements that do not exist
// stay undefined, and are not used).
template <typename T>
__device__ __forceinline__ void load_rows(const T *src, T (&val)[kRowPass], const RowMap &m, int u0,
                                          const CONST_AS BiasPass &ps) {
    const char *sb = (const char *)src;
    constexpr uint32_t es = sizeof(T);
    const uint32_t gap = (uint32_t)(ps.sv - ps.nu * ps.su);   // from a plane's last row to the next plane's first
    if (m.whole && m.nval <= ps.nu) {   // at most two planes
        const uint32_t vo = (uint32_t)(m.sub * ps.su + m.col) * es;
        const int cross = ps.nu - u0 - m.sub;   // this lane's rows from here on lie in the second
        int r = 0;
        m.each((uint32_t)ps.su * es, [&](int i, uint32_t at) {
            val[i] = *(const T *)(sb + (vo + at + (r >= cross ? gap * es : 0u)));
            r += 1 << m.lgr;
        });
    } else {
        // plane of row r: floor((u0 + r) / nu), exact in FP32 for these few rows
        const float inv = 1.0f / (float)ps.nu;
        m.any([&](int i, int r, int c) {
            const uint32_t q = (uint32_t)(((float)(u0 + r) + 0.5f) * inv);
            val[i] = *(const T *)(sb + ((uint32_t)(r * ps.su + c) + q * gap) * es);
        });
    }
}
// ... and from val into the wave's tile.
template <typename T>
__device__ __forceinline__ void put_rows(T *tile, const T (&val)[kRowPass], const RowMap &m, int pitch) {
    if (m.whole) {
        T *t = tile + m.sub * pitch + m.col;
        m.each(pitch, [&](int i, int at) { t[at] = val[i]; });
    } else {
        m.any([&](int i, int r, int c) { tile[r * pitch + c] = val[i]; });
    }
    wave_sync();
}
// ... and from the tile to consecutive rows of cols elements.
template <typename T>
__device__ __forceinline__ void drain_rows(T *dst, const T *tile, const RowMap &m, int pitch) {
    constexpr uint32_t es = sizeof(T);
    if (m.whole) {
        const T *t = tile + m.sub * pitch + m.col;
        const uint32_t vo = (uint32_t)(m.sub * m.cols + m.col) * es;
        T val[kRowPass];
        m.each(pitch, [&](int i, int at) { val[i] = t[at]; });
        m.each((uint32_t)m.cols * es,
               [&](int i, uint32_t at) { __builtin_nontemporal_store(val[i], (T *)((char *)dst + (vo + at))); });
    } else {
        m.any([&](int i, int r, int c) {
            __builtin_nontemporal_store(tile[r * pitch + c], (T *)((char *)dst + (uint32_t)(r * m.cols + c) * es));
        });
    }
}

// Rows of more than 64 columns, in the WIDE kernels: column blocks of 64, every
// row's first block, then every row's second, where RowMap's general walk, with
// masks and a plane search in every pass, is what bounds them: x lines of 80
// nodes, 5 fields of 80 x 96 x 96, X_2 pair, FP64 36.7 -> 26.5 us, FP32 33.0 -> 18.0
// (96 nodes: 37.6 -> 28.2, 33.1 -> 18.5).  They are kernels of their own: in one
// kernel the second form of the row moves costs rows of one block up to a tenth.
struct WideMap {
    int cols, nval, lgr;   // columns, real rows, log2 of rows per pass
    int sub, col;          // this lane's row in a pass and column
    int npass;
    int lgg;               // log2 of a column block's passes / 4
    bool whole;            // passes in groups of four, every row real, loaded from at most two planes (put_rows
                           // stores every lane's value, so load_rows must have loaded it)
    __device__ __forceinline__ WideMap(int cols_, int nval_, int NW, int lane, int nu) : cols(cols_), nval(nval_) {
        lgr = cols > 32 ? 0 : cols > 16 ? 1 : 2;
        sub = lane >> (6 - lgr);
        col = lane & ((64 >> lgr) - 1);
        npass = (NW >> lgr) * ((cols + 63) >> 6);
        const int rp = NW >> lgr;   // passes of a column block
        lgg = rp >= 16 ? 2 : rp >= 8 ? 1 : 0;
        whole = nval == NW && rp >= 4 && nval <= nu;
    }
    // Whole maps: fn(i, r, at): in pass i this lane's element lies r rows below
    // its first one and at (rows of step, columns of unit) from the first row's
    // first.  Lanes past the last column take that column once more:
    // they load and store what its own lane does, and no pass is masked.
    template <typename U, typename Fn>
    __device__ __forceinline__ void each(U step, U unit, Fn fn) const {
#pragma unroll
        for (int g = 0; g < kRowPass / 4; ++g)
            if (4 * g < npass) {
                const int blk = g >> lgg, r0 = ((g - (blk << lgg)) << 2) << lgr;
                const U c = (U)sub * step + (U)min(col + 64 * blk, cols - 1) * unit;
                U at = (U)r0 * step;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    fn(4 * g + i, r0 + (i << lgr), c + at);
                    at += step << lgr;
                }
            }
    }
    // Any map: fn(i, row, column) for the elements that exist.
    template <typename Fn>
    __device__ __forceinline__ void any(Fn fn) const {
        int r = 0, c = 0;
#pragma unroll
        for (int i = 0; i < kRowPass; ++i)
            if (i < npass) {
                if (c + col < cols && r + sub < nval) fn(i, r + sub, c + col);
                const bool last = c + 64 >= cols;
                r += last ? 1 << lgr : 0;
                c = last ? 0 : c + 64;
            }
    }
};
// Rows from src (the first line's column 0; the first line is row u0 of its
// plane) into val, all requested before any is used (elements that do not exist
// stay undefined, and are not used).
template <typename T>
__device__ __forceinline__ void load_rows(const T *src, T (&val)[kRowPass], const WideMap &m, int u0,
                                          const CONST_AS BiasPass &ps) {
    const char *sb = (const char *)src;
    constexpr uint32_t es = sizeof(T);
    const uint32_t gap = (uint32_t)(ps.sv - ps.nu * ps.su);   // from a plane's last row to the next plane's first
    if (m.whole) {   // at most two planes
        const int cross = ps.nu - u0 - m.sub;   // this lane's rows from here on lie in the second
        m.each((uint32_t)ps.su * es, es, [&](int i, int r, uint32_t at) {
            val[i] = *(const T *)(sb + (at + (r >= cross ? gap * es : 0u)));
        });
    } else {
        // plane of row r: floor((u0 + r) / nu), exact in FP32 for these few rows
        const float inv = 1.0f / (float)ps.nu;
        m.any([&](int i, int r, int c) {
            const uint32_t q = (uint32_t)(((float)(u0 + r) + 0.5f) * inv);
            val[i] = *(const T *)(sb + ((uint32_t)(r * ps.su + c) + q * gap) * es);
        });
    }
}
// ... and from val into the wave's tile.
template <typename T>
__device__ __forceinline__ void put_rows(T *tile, const T (&val)[kRowPass], const WideMap &m, int pitch) {
    if (m.whole) {
        m.each(pitch, 1, [&](int i, int, int at) { tile[at] = val[i]; });
    } else {
        m.any([&](int i, int r, int c) { tile[r * pitch + c] = val[i]; });
    }
    wave_sync();
}
// ... and from the tile to consecutive rows of cols elements.
template <typename T>
__device__ __forceinline__ void drain_rows(T *dst, const T *tile, const WideMap &m, int pitch) {
    constexpr uint32_t es = sizeof(T);
    if (m.whole) {
        T val[kRowPass];
        m.each(pitch, 1, [&](int i, int, int at) { val[i] = tile[at]; });
        m.each((uint32_t)m.cols * es, es,
               [&](int i, int, uint32_t at) { __builtin_nontemporal_store(val[i], (T *)((char *)dst + at)); });
    } else {
        m.any([&](int i, int r, int c) {
            __builtin_nontemporal_store(tile[r * pitch + c], (T *)((char *)dst + (uint32_t)(r * m.cols + c) * es));
        });
    }
}

template <bool WIDE>
__device__ __forceinline__ auto row_map(int cols, int nval, int NW, int lane, int nu) {
    if constexpr (WIDE)
        return WideMap(cols, nval, NW, lane, nu);
    else
        return RowMap(cols, nval, NW, lane);
}

// One wave: NW = 64 / P lines of one field of one pass, P = 2^lgP partitions
// per line (lane = p NW + line).  N = P (L - 1) + nfull: the first nfull
// partitions hold L rows, the others L - 1, so only row L - 1 differs between
// lanes.  Iterated closures (Eq. iter_left_X and its mirror; ev given): every
// row of a closure line takes the interior scheme, and the solution entering at
// node -1 (left bias) / N (right bias) is ev[2 e] / ev[2 e + 1] of the line's
// entry e = ev_base + field * nlines + line, instead of the closure rows.  ends
// (if given) receives, unscaled (before h^-1), the left-biased solution at node
// N - 1 and the right-biased one at node 0 of every line, the values the
// neighbours' next iterate enters with.  Off: byte offsets of a lane's line
// relative to the wave's first line (32 bits where they fit).
template <typename T, int HB, bool EMB, bool WIDE, int L, typename Off>
__device__ __forceinline__ void bias_wave(const CONST_AS BiasPass *pass, int field, int line0, int lgP, int tilew,
                                          const T *__restrict__ coefs, const T *__restrict__ in, T *__restrict__ out,
                                          const T *__restrict__ ev, T *__restrict__ ends, T *smem) {
    constexpr int W = L + 2 * HB;   // f[t] = node k0 - HB + t
    const CONST_AS BiasPass &ps = *pass;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int P = 1 << lgP, lgN = 6 - lgP, NW = 64 >> lgP;
    const int N = ps.N;
    int first = line0 + wv * NW;   // this wave's first line
    if (first >= ps.nlines) return;
    // the last wave of a pass takes whole NW lines too, some of them also the
    // wave's before it (both store the same values)
    first = max(0, min(first, ps.nlines - NW));
    const int nfull = N - P * (L - 1);
    const int p = lane >> lgN, l = lane & (NW - 1);
    const bool full = p < nfull, islast = p == P - 1;
    const bool lastfull = nfull == P;
    const int k0 = p * (L - 1) + min(p, nfull);
    int line = first + l;
    const bool active = line < ps.nlines;
    if (!active) line = ps.nlines - 1;
    const int v0 = __builtin_amdgcn_readfirstlane(first / ps.nu), u0 = first - v0 * ps.nu;
    const int v = line / ps.nu, u = line - v * ps.nu;
    const bool xdir = ps.sd == 1;
    const bool periodic = ps.periodic;
    const bool iter = ev != nullptr && !periodic;
    const bool closed = !periodic && !iter;
    const int mode = ps.mode;
    const bool left = mode <= 0 || mode == 2;   // -1 left, 0 upwind, 1 right, 2 symmetrised
    const bool right = mode >= 0;
    const CONST_AS T *rec = (const CONST_AS T *)coefs + (int64_t)ps.tab * kBiasRec;
    const T alpha = rec[0], inv_det = rec[24];
    T *tile = smem + (int64_t)wv * tilew;

    const int64_t base0 = (int64_t)u0 * ps.su + (int64_t)v0 * ps.sv;   // the wave's first line in a field
    const int64_t fbase = ps.in_base + (int64_t)field * ps.in_fstride + base0;
    const int64_t sdB = (int64_t)ps.sd * (int64_t)sizeof(T);
    const int64_t lineoff = (int64_t)u * ps.su + (int64_t)v * ps.sv - base0;
    const Off voff = (Off)((lineoff + (int64_t)k0 * ps.sd) * (int64_t)sizeof(T));
    const int nval = min(NW, ps.nlines - first);   // real lines of this wave

    // ---- partition rows and halo into registers; nodes outside the stored line
    // (a class wider than the scheme, or the missing row of the last partition)
    // read as 0
    T f[W];
    T *trow;   // x lines: this lane's rows in the tile of N columns
    if (xdir) {
        const int e = bias_ghosts(ps.ng, HB, periodic);
        const int Tn = N + 2 * e, tp = Tn | 1;
        {
            T raw[kRowPass];
            const auto m = row_map<WIDE>(Tn, nval, NW, lane, ps.nu);
            load_rows(in + fbase - e, raw, m, u0, ps);
            put_rows(tile, raw, m, tp);
        }
        if (periodic) {
            const T *row = tile + l * tp;
            int j = (k0 - HB) % N;
            j += j < 0 ? N : 0;
#pragma unroll
            for (int t = 0; t < W; ++t) {
                f[t] = row[j];
                ++j;
                j = j == N ? 0 : j;
            }
        } else {
            const T *row = tile + l * tp + k0 + (e - HB);
            if (e > HB || (e == HB && lastfull)) {
#pragma unroll
                for (int t = 0; t < W; ++t) f[t] = row[t];
            } else {
#pragma unroll
                for (int t = 0; t < W; ++t) {
                    const int j = k0 - HB + t;
                    f[t] = T(0);
                    if (j >= -e && j < N + e) f[t] = row[t];
                }
            }
        }
        wave_sync();   // the tile is reused for the velocity and the output
        trow = tile + l * (N | 1) + k0;
    } else if (periodic) {
        const char *src = (const char *)(in + fbase);
        const Off lo = (Off)(lineoff * (int64_t)sizeof(T));
        int j = (k0 - HB) % N;
        j += j < 0 ? N : 0;
#pragma unroll
        for (int t = 0; t < W; ++t) {
            f[t] = *(const T *)(src + (Off)(lo + (Off)j * (Off)sdB));
            ++j;
            j = j == N ? 0 : j;
        }
    } else {
        const char *src = (const char *)(in + fbase) - HB * sdB;
        if (ps.ng > HB || (ps.ng == HB && lastfull)) {
#pragma unroll
            for (int t = 0; t < W; ++t) {
                f[t] = *(const T *)(src + voff);
                src = later(src + sdB);
            }
        } else {
#pragma unroll
            for (int t = 0; t < W; ++t) {
                const int j = k0 - HB + t;
                f[t] = T(0);
                if (j >= -ps.ng && j < N + ps.ng) f[t] = *(const T *)(src + voff);
                src += sdB;
            }
        }
    }

    // Scans over a line's partitions: v, the value leaving a partition for a zero
    // value entering it, becomes the one for a zero value entering the line; w,
    // the weight of the entering value, (-alpha)^rows.
    auto scan_up = [&](T vv, T w) {
        for (int s = 1; s < P; s <<= 1) {
            const T t = __shfl(vv, lane - s * NW), tw = __shfl(w, lane - s * NW);
            if (p >= s) {
                vv += w * t;
                w *= tw;
            }
        }
        return vv;
    };
    auto scan_down = [&](T vv, T w) {
        for (int s = 1; s < P; s <<= 1) {
            const T t = __shfl(vv, lane + s * NW), tw = __shfl(w, lane + s * NW);
            if (p + s < P) {
                vv += w * t;
                w *= tw;
            }
        }
        return vv;
    };
    const int lastlane = (P - 1) * NW + l;

    // ---- right-hand sides (closure rows where this lane holds them); window of
    // row i: f[i + HB + m] is node k0 + i + m
    const bool closureL = closed && p == 0;
    const bool closureR = closed && islast;
    T rl[L], rr[L];
    T s2v[EMB ? L : 1];
    if constexpr (EMB) {
        // W: the compact second derivative (2)P1_M on the same rows, explicit
        // closure rows.  [a2, 1, a2] = (1 + b S-)(1 + b S+) a2 / b on the infinite
        // line, so it is a forward and a backward recurrence over the line with
        // zero right side on the closure rows, whose values are then met with
        // the two homogeneous solutions (-b)^k, (-b)^(N-1-k).
        const T beta = rec[25], ibeta = rec[28];
        const CONST_AS T *pb = rec + kBiasPow2;   // (-beta)^n
        T (&s)[L] = s2v;
        T e0 = T(0), e1 = T(0);
        {
            const CONST_AS T *st = rec + kBiasSt2;
            constexpr int M2 = HB - 2;   // W_M: classes M + 2, (2)P1_M of half-width M
#pragma unroll
            for (int i = 0; i < L; ++i) {
                T r = st[5] * f[i + HB];
#pragma unroll
                for (int m = 1; m <= M2; ++m) r += st[5 + m] * (f[i + HB + m] + f[i + HB - m]);
                s[i] = r;
            }
        }
        if (closed) {
            const CONST_AS T *sc = rec + kBiasCl2;
#pragma unroll
            for (int m = -HB; m <= HB; ++m) e0 += sc[5 + m] * f[HB + m];
            if (p == 0) s[0] = T(0);
            if (lastfull) {
#pragma unroll
                for (int m = -HB; m <= HB; ++m) e1 += sc[5 - m] * f[L - 1 + HB + m];
                if (islast) s[L - 1] = T(0);
            } else if constexpr (L >= 2) {
#pragma unroll
                for (int m = -HB; m <= HB; ++m) e1 += sc[5 - m] * f[L - 2 + HB + m];
                if (islast) s[L - 2] = T(0);
            }
        }
        {
#pragma unroll
            for (int i = 1; i < L; ++i) s[i] -= beta * s[i - 1];
            const T uE = full ? s[L - 1] : s[L - 2];
            const T w = full ? pb[L] : pb[L - 1];
            T U = __shfl(scan_up(uE, w), lane - NW);
            if (p == 0) U = T(0);
            if (periodic) U += pb[k0] * (__shfl(uE + w * U, lastlane) * (T)ps.wrap2);
#pragma unroll
            for (int i = 0; i < L; ++i) s[i] += pb[i + 1] * U;
        }
        if (!full) s[L - 1] = T(0);
#pragma unroll
        for (int i = L - 2; i >= 0; --i) s[i] -= beta * s[i + 1];
        const T vS = scan_down(s[0], full ? pb[L] : pb[L - 1]);
        T S = __shfl(vS, lane + NW);
        if (islast) S = T(0);
        const int up = N - k0 - (full ? L : L - 1);   // rows above this partition
        T K1 = T(0), K2 = T(0);
        if (periodic) {
            S += pb[up] * (__shfl(vS, l) * (T)ps.wrap2);
        } else {
            const T d0 = __shfl(e0, l) - __shfl(vS, l);
            const T d1 = __shfl(e1, lastlane) - __shfl(lastfull ? s[L - 1] : s[L - 2], lastlane);
            const T bN = pb[N - 1];
            K1 = (d0 - bN * d1) * (T)ps.det2 * pb[k0];
            K2 = (d1 - bN * d0) * (T)ps.det2 * pb[up];
        }
        K2 -= beta * S;
        if (!full) K2 *= ibeta;   // weights below count from row L - 1
#pragma unroll
        for (int i = 0; i < L; ++i) s[i] += K1 * pb[i] + K2 * pb[L - 1 - i];
        __builtin_amdgcn_sched_barrier(0);   // s before the biases' sides: fewer rows live at once
    }
    {
        const CONST_AS T *ac = later(rec) + 1 + kBiasHalf;
        constexpr int MI = EMB ? HB - 1 : HB;   // W_M: interior half-width M + 1
        T a[2 * MI + 1];
#pragma unroll
        for (int m = -MI; m <= MI; ++m) a[m + MI] = ac[m];
#pragma unroll
        for (int i = 0; i < L; ++i) {
            T x = T(0), y = T(0);
            if constexpr (EMB) {
                x = s2v[i];
                y = -s2v[i];
            }
#pragma unroll
            for (int m = -MI; m <= MI; ++m) {
                x += a[m + MI] * f[i + HB + m];
                y -= a[m + MI] * f[i + HB - m];
            }
            rl[i] = x;
            rr[i] = y;
        }
    }
    if (!EMB && ps.s2_in) {   // U: the sampled second derivative
        const T *s2 = in + ps.s2_base + (int64_t)u * ps.s2u + (int64_t)v * ps.s2v + (int64_t)k0 * ps.s2d;
        const T w2 = (T)ps.w2;
#pragma unroll
        for (int i = 0; i < L; ++i)
            if (i < L - 1 || full) {
                const T e = w2 * s2[(int64_t)i * ps.s2d];
                rl[i] += e;
                rr[i] -= e;
            }
    }
    if (closed) {
        const CONST_AS T *c = rec + 12 + kBiasHalf;
        T e0 = T(0), e1 = T(0);
        if (!EMB && ps.s2_in) {
            const T *s2 = in + ps.s2_base + (int64_t)u * ps.s2u + (int64_t)v * ps.s2v;
            e0 = (T)ps.w2c * s2[0];
            e1 = (T)ps.w2c * s2[(int64_t)(N - 1) * ps.s2d];
        }
#pragma unroll
        for (int m = -HB; m <= HB + 1; ++m) e0 += c[m] * f[HB + m];
        if (closureL) rl[0] = e0;
        if (lastfull) {
#pragma unroll
            for (int m = -HB; m <= HB + 1; ++m) e1 += c[m] * f[L - 1 + HB - m];
            if (closureR) rr[L - 1] = -e1;
        } else if constexpr (L >= 3) {
#pragma unroll
            for (int m = -HB; m <= HB + 1; ++m) e1 += c[m] * f[L - 2 + HB - m];
            if (closureR) rr[L - 2] = -e1;
        }
    }

    // The velocity, requested once the window is dead and before the solves and
    // scans that its latency overlaps: rows k0 .. k0 + L - 1 of y and z lines,
    // whole rows of x lines, put into order through the tile below.
    T c[L < kRowPass ? kRowPass : L];
    if (mode == 0) {
        if (xdir) {
            load_rows(in + ps.vel_base + base0, c, row_map<WIDE>(N, nval, NW, lane, ps.nu), u0, ps);
        } else {
            const char *vl = (const char *)(in + ps.vel_base + base0);
#pragma unroll
            for (int i = 0; i < L - 1; ++i) {
                c[i] = *(const T *)(vl + voff);
                vl = later(vl + sdB);
            }
            c[L - 1] = T(0);
            if (full) c[L - 1] = *(const T *)(vl + voff);
        }
        __builtin_amdgcn_sched_barrier(0);
    }

    // ---- local solves with zero entering values
    T xE = T(0);   // left bias: the value leaving the partition
    if (left) {
        if (closureL) rl[0] = (rl[0] - alpha * rl[1]) * inv_det;
#pragma unroll
        for (int i = 1; i < L; ++i) rl[i] -= alpha * rl[i - 1];
        xE = full ? rl[L - 1] : rl[L - 2];
    }
    if (right) {
        if (closureR) {
            if (lastfull) rr[L - 1] = (rr[L - 1] - alpha * rr[L - 2]) * inv_det;
            else if constexpr (L >= 3) rr[L - 2] = (rr[L - 2] - alpha * rr[L - 3]) * inv_det;
        }
        if (!full) rr[L - 1] = T(0);
#pragma unroll
        for (int i = L - 2; i >= 0; --i) rr[i] -= alpha * rr[i + 1];
    }
    const CONST_AS BiasPass &pt = *later(pass);
    const CONST_AS T *pw = later(rec) + kBiasPow;   // (-alpha)^n
    // ---- true values entering the partition
    T X = T(0), Y = T(0);
    const T wP = full ? pw[L] : pw[L - 1];
    const int64_t eix = 2 * (pt.ev_base + (int64_t)field * pt.nlines + line);   // this line's end entries
    if (left) {
        X = __shfl(scan_up(xE, wP), lane - NW);
        if (p == 0) X = T(0);
        if (periodic) X += rec[kBiasPow + k0] * (__shfl(xE + wP * X, lastlane) * (T)pt.wrap);
        if (iter) X += rec[kBiasPow + k0] * ev[eix];
        if (ends && !periodic && active && islast) ends[eix] = xE + wP * X;
    }
    if (right) {
        const T vR = scan_down(rr[0], wP);
        Y = __shfl(vR, lane + NW);
        if (islast) Y = T(0);
        const int up = N - k0 - (full ? L : L - 1);   // rows above this partition
        if (periodic) Y += rec[kBiasPow + up] * (__shfl(vR, l) * (T)pt.wrap);
        if (iter) Y += rec[kBiasPow + up] * ev[eix + 1];
        if (ends && !periodic && active && p == 0) ends[eix + 1] = rr[0] + wP * Y;
        if (!full) Y *= rec[27];   // -1 / alpha: the weights below count from row L
    }

    // ---- corrected values, combined and stored
    const T hinv = (T)pt.hinv;
    if (mode == 0) {
        if (xdir) {
            put_rows(tile, c, row_map<WIDE>(N, nval, NW, lane, pt.nu), N | 1);
#pragma unroll
            for (int i = 0; i < L; ++i) c[i] = trow[i];
        }
#pragma unroll
        for (int i = 0; i < L; ++i) {
            const T xL = rl[i] + pw[i + 1] * X;
            const T xR = rr[i] + pw[L - i] * Y;
            const T ch = c[i] * hinv;
            rl[i] = fmin(ch, (T)0) * xR + fmax(ch, (T)0) * xL;
        }
    } else if (mode < 0) {
#pragma unroll
        for (int i = 0; i < L; ++i) rl[i] = hinv * (rl[i] + pw[i + 1] * X);
    } else if (mode == 1) {
#pragma unroll
        for (int i = 0; i < L; ++i) rl[i] = hinv * (rr[i] + pw[L - i] * Y);
    } else {
#pragma unroll
        for (int i = 0; i < L; ++i)
            rl[i] = T(0.5) * (hinv * (rl[i] + pw[i + 1] * X) + hinv * (rr[i] + pw[L - i] * Y));
    }
    T *o = out + pt.out_base + (int64_t)field * pt.out_fstride;
    if (xdir) {   // the rows of consecutive x lines are contiguous in the output
#pragma unroll
        for (int i = 0; i < L - 1; ++i) trow[i] = rl[i];
        if (full) trow[L - 1] = rl[L - 1];
        wave_sync();
        drain_rows(o + (int64_t)first * N, tile, row_map<WIDE>(N, nval, NW, lane, INT_MAX), N | 1);
    } else if (active) {
        const int64_t obase0 = (int64_t)u0 * pt.osu + (int64_t)v0 * pt.osv;
        const int64_t osdB = (int64_t)pt.osd * (int64_t)sizeof(T);
        char *dst = (char *)(o + obase0);
        const Off ovoff =
            (Off)(((int64_t)u * pt.osu + (int64_t)v * pt.osv - obase0 + (int64_t)k0 * pt.osd) * (int64_t)sizeof(T));
        // Runs of less than 64 bytes meet their neighbours' in the L2: 97 nodes of y,
        // 5 fields, 40.7 -> 37.2 us FP64, 34.6 -> 29.8 FP32, where shorter lines lose (48
        // nodes, FP32: 9.0 -> 10.1).  Only in the WIDE kernels: the second store loop alone costs the
        // narrow FP32 kernel 6 %.
        if (!WIDE || NW * (int)sizeof(T) >= 64) {
#pragma unroll
            for (int i = 0; i < L - 1; ++i) {
                __builtin_nontemporal_store(rl[i], (T *)(dst + ovoff));
                dst = later(dst + osdB);
            }
            if (full) __builtin_nontemporal_store(rl[L - 1], (T *)(dst + ovoff));
        } else {
#pragma unroll
            for (int i = 0; i < L - 1; ++i) {
                *(T *)(dst + ovoff) = rl[i];
                dst = later(dst + osdB);
            }
            if (full) *(T *)(dst + ovoff) = rl[L - 1];
        }
    }
}

template <typename T, int HB, bool EMB, bool WIDE, typename Off, int L0, int... Ls>
__device__ __forceinline__ void bias_dispatch(int L, const CONST_AS BiasPass *ps, int field, int line0, int lgP, int tilew,
                                              const T *coefs, const T *in, T *out, const T *ev, T *ends, T *smem) {
    if (L == L0) {
        bias_wave<T, HB, EMB, WIDE, L0, Off>(ps, field, line0, lgP, tilew, coefs, in, out, ev, ends, smem);
        return;
    }
    if constexpr (sizeof...(Ls) > 0)
        bias_dispatch<T, HB, EMB, WIDE, Off, Ls...>(L, ps, field, line0, lgP, tilew, coefs, in, out, ev, ends, smem);
}

// Waves per SIMD the registers are held to.  FP64 with 12 rows: 128 registers
// (4 waves) hold a pair of biases without spills; 64 blocks, 22 fields, X_2
// pair: 463 us, with partitions of at most 8 rows and 5 waves 560 us (the halo
// doubles the loads).  With an embedded second derivative FP64 takes 2 waves
// (739 us; 3 waves spill: 1331 us), FP32 4 (354 us; 3 waves 390 us).
#define BIAS_WPE(T, EMB) (sizeof(T) == 8 ? (EMB ? 2 : 4) : (EMB ? 4 : 6))
// Work item meta: lgP in bits 0..3, L in bits 4..11.  tilew: elements of one
// wave's tile.
template <typename T, int HB, bool EMB, bool WIDE, typename Off, int... Ls>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(BIAS_WPE(T, EMB)))) void k_biased_wave(const BiasItem *__restrict__ items,
                                                     const BiasPass *__restrict__ passes,
                                                     const T *__restrict__ coefs, const T *__restrict__ in,
                                                     T *__restrict__ out, const T *__restrict__ ev,
                                                     T *__restrict__ ends, int tilew) {
    extern __shared__ __align__(16) unsigned char smem[];
    const BiasItem item = items[blockIdx.x];
    if (item.pass < 0) return;   // padding of the XCD-interleaved order (whole workgroup)
    bias_dispatch<T, HB, EMB, WIDE, Off, Ls...>(item.meta >> 4, (const CONST_AS BiasPass *)passes + item.pass, item.field, item.line0, item.meta & 15,
                                          tilew, coefs, in, out, ev, ends, (T *)smem);
}

// Partition lengths compiled into every instance.
#define BIAS_LS 12, 8, 11, 10, 9, 7, 6, 5, 4, 3, 2

// The instances of one element type and row moves or offsets: per half-width
// class, with or without an embedded second derivative (half-widths 3 .. 5).
// Off uint64_t: fields of 4 GiB and more, which have no WIDE kernel.
template <typename T, bool WIDE, typename Off>
const void *wave_fn(int hb, int emb) {
    if (emb) switch (hb) {
            case 3: return (const void *)k_biased_wave<T, 3, true, WIDE, Off, BIAS_LS>;
            case 4: return (const void *)k_biased_wave<T, 4, true, WIDE, Off, BIAS_LS>;
            case 5: return (const void *)k_biased_wave<T, 5, true, WIDE, Off, BIAS_LS>;
            default: return nullptr;
        }
    switch (hb) {
        case 2: return (const void *)k_biased_wave<T, 2, false, WIDE, Off, BIAS_LS>;
        case 3: return (const void *)k_biased_wave<T, 3, false, WIDE, Off, BIAS_LS>;
        case 4: return (const void *)k_biased_wave<T, 4, false, WIDE, Off, BIAS_LS>;
        case 5: return (const void *)k_biased_wave<T, 5, false, WIDE, Off, BIAS_LS>;
        default: return nullptr;
    }
}

}  // namespace
}  // namespace cfd
