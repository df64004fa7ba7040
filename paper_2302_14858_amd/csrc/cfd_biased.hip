// Biased (upwind) compact first derivatives on the lines of mesh blocks
// (arXiv 2302.14858, Sec. ssec:domdec_drp).
//
// Left-biased rows: alpha x_{k-1} + x_k = sum_m a_m f_{k+m} (k > k*_-), with
// the closure row x_{k*_-} + alpha x_{k*_- + 1} = sum_m c_m f_{k*_- + m}
// (Eq. closure_left_X).  The right-biased operator is the mirror image:
// x_k + alpha x_{k+1} = -sum_m a_{-m} f_{k+m} (k < k*_+), closure row
// alpha x_{k*_+ - 1} + x_{k*_+} = -sum_m c_{-m} f_{k*_+ + m}.  Each system is
// bidiagonal apart from its closure row, so the two rows at the closed end
// are solved together and the rest is one recurrence away from that end.
// On periodic lines every row is an interior row with indices taken modulo N;
// the cyclic recurrence is closed by its wrap value
//   x^L_{N-1} = sum_j (-alpha)^(N-1-j) r^L_j / (1 - (-alpha)^N),
//   x^R_0     = sum_j (-alpha)^j r^R_j       / (1 - (-alpha)^N),
// both accumulated in one forward pre-sweep.
//
// Upwind operator (Eq. biasderapproxadv, with c the velocity field sampled on
// the grid): c d f = min(c, 0) D[right] f + max(c, 0) D[left] f.
//
// W schemes (Tab. ccuw_deg_one_col) add w2 s_k to every interior row's right
// side (-w2 s_k for the right bias), s the embedded second derivative of unit
// spacing and w2 = a2; the closure rows take none.
// U schemes (Tab. ucd_slow) read s, the sampled f'', from an input field and
// add it on every row, the closure row with its own weight w2c.
//
// Wave kernel (x lines of up to 1024 nodes, y and z lines of up to 256): a
// wave owns 64 / P lines of one field, P = 1 .. 64 a power of two, and its
// lanes are the P partitions of those lines (lane = partition * (64 / P) +
// line, at most 8, 12 or 16 rows each).  A lane issues every load of its rows
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
//
// Sweep kernel (longer y and z lines): one lane per line, a register window of
// 2 HB + 3 samples slid one node per row; the right-biased sweep leaves
// min(c,0) D[right] f in the output, the left-biased sweep adds the rest.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "cfd_internal.h"

namespace cfd {
namespace {

template <typename T>
struct BLine {
    const T *f;
    int64_t sd;
    int N, ng, periodic;
    __device__ __forceinline__ T ld(int j) const {
        if (periodic) {
            j %= N;
            if (j < 0) j += N;
            return f[(int64_t)j * sd];
        }
        return (j >= -ng && j < N + ng) ? f[(int64_t)j * sd] : T(0);
    }
};

template <typename T, int HB>
struct BCoef {
    T alpha, inv_det;
    T a[2 * HB + 1];   // a_{-HB..HB}
    T c[2 * HB + 2];   // c_{-HB..HB+1}
};

// window index of offset m: HB + 1 + m
template <typename T, int HB>
__device__ __forceinline__ T left_interior(const BCoef<T, HB> &q, const T *w) {
    T r = 0;
#pragma unroll
    for (int m = -HB; m <= HB; ++m) r += q.a[m + HB] * w[HB + 1 + m];
    return r;
}
template <typename T, int HB>
__device__ __forceinline__ T left_closure(const BCoef<T, HB> &q, const T *w) {
    T r = 0;
#pragma unroll
    for (int m = -HB; m <= HB + 1; ++m) r += q.c[m + HB] * w[HB + 1 + m];
    return r;
}
template <typename T, int HB>
__device__ __forceinline__ T right_interior(const BCoef<T, HB> &q, const T *w) {
    T r = 0;
#pragma unroll
    for (int m = -HB; m <= HB; ++m) r -= q.a[m + HB] * w[HB + 1 - m];
    return r;
}
template <typename T, int HB>
__device__ __forceinline__ T right_closure(const BCoef<T, HB> &q, const T *w) {
    T r = 0;
#pragma unroll
    for (int m = -HB; m <= HB + 1; ++m) r -= q.c[m + HB] * w[HB + 1 - m];
    return r;
}

template <typename T, int HB>
__device__ __forceinline__ void load_coef(BCoef<T, HB> &q, const T *rec) {
    q.alpha = rec[0];
    q.inv_det = rec[24];
#pragma unroll
    for (int m = -HB; m <= HB; ++m) q.a[m + HB] = rec[1 + kBiasHalf + m];
#pragma unroll
    for (int m = -HB; m <= HB + 1; ++m) q.c[m + HB] = rec[12 + kBiasHalf + m];
}

// Orders the LDS accesses of one wave (its LDS operations execute in order, so
// only the compiler has to keep them so); no other wave shares the tile.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Walk of a lane over the elements e = lane, lane + 64, ... of the [lines][cols]
// rows of a wave's x lines, in row-major order: the row and column, and the
// element's offset in a field (the caller's dq = 64 / cols and dr = 64 % cols
// step it without a division).
struct RowWalk {
    int r, j, uu;
    int64_t off;
    __device__ __forceinline__ RowWalk(int lane, int cols, int line0, int t0, const BiasPass &ps) {
        r = lane / cols;
        j = lane - r * cols;
        const int ln = line0 + r;
        const int vv = ln / ps.nu;
        uu = ln - vv * ps.nu;
        off = (int64_t)uu * ps.su + (int64_t)vv * ps.sv + t0 + j;
    }
    __device__ __forceinline__ void next(int cols, int dq, int dr, const BiasPass &ps) {
        int dl = dq;
        j += dr;
        off += dr;
        if (j >= cols) {
            j -= cols;
            off -= cols;
            ++dl;
        }
        r += dl;
        uu += dl;
        off += (int64_t)dl * ps.su;
        while (uu >= ps.nu) {
            uu -= ps.nu;
            off += (int64_t)ps.sv - (int64_t)ps.nu * ps.su;
        }
    }
};

// One wave: NW = 64 / P lines of one field of one pass, P = 2^lgP partitions of
// Lr <= L rows per line (lane = p NW + line), Pu of them holding rows.  Iterated
// closures (Eq. iter_left_X and its mirror; ev given): every row of a closure
// line takes the interior scheme, and the solution entering at node -1 (left
// bias) / N (right bias) is ev[2 e] / ev[2 e + 1] of the line's entry e =
// ev_base + field * nlines + line, instead of the closure rows.  ends (if
// given) receives, unscaled (before h^-1), the left-biased solution at node
// N - 1 and the right-biased one at node 0 of every line, the values the
// neighbours' next iterate enters with.  Off: byte offsets of a lane's line
// relative to the item's first line (32 bits where they fit).
template <typename T, int HB, bool EMB, int L, typename Off>
__device__ __forceinline__ void bias_wave(const BiasPass &ps, int field, int line0, int lgP, int Lr, int tilew,
                                          const T *__restrict__ coefs, const T *__restrict__ in, T *__restrict__ out,
                                          const T *__restrict__ ev, T *__restrict__ ends, T *smem) {
    constexpr int W = L + 2 * HB + 2;   // f[i] = node k0 - HB - 1 + i
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int P = 1 << lgP, lgN = 6 - lgP, NW = 64 >> lgP;
    const int N = ps.N;
    const int first = line0 + wv * NW;   // this wave's first line
    if (first >= ps.nlines) return;
    const int Pu = (N + Lr - 1) / Lr, nlast = N - (Pu - 1) * Lr;   // >= 2 (host)
    const int p = lane >> lgN, l = lane & (NW - 1);
    const bool idle = p >= Pu, islast = p == Pu - 1;
    const int k0 = idle ? 0 : p * Lr;    // idle lanes read partition 0 and take no part
    int line = first + l;
    const bool active = line < ps.nlines;
    if (!active) line = ps.nlines - 1;
    const int v0 = first / ps.nu, u0 = first - v0 * ps.nu;
    const int v = line / ps.nu, u = line - v * ps.nu;
    const bool xdir = ps.sd == 1;
    const bool periodic = ps.periodic;
    const bool iter = ev != nullptr && !periodic;
    const bool closed = !periodic && !iter;
    const int mode = ps.mode;
    const bool left = mode <= 0 || mode == 2;   // -1 left, 0 upwind, 1 right, 2 symmetrised
    const bool right = mode >= 0;
    const T *rec = coefs + (int64_t)ps.tab * kBiasRec;
    BCoef<T, HB> q;
    load_coef<T, HB>(q, rec);
    const T alpha = q.alpha;
    const T *pw = rec + kBiasPow;   // (-alpha)^n
    T *tile = smem + (int64_t)wv * tilew;

    const int64_t base0 = (int64_t)u0 * ps.su + (int64_t)v0 * ps.sv;   // the wave's first line in a field
    const int64_t fbase = ps.in_base + (int64_t)field * ps.in_fstride;
    const int64_t sdB = (int64_t)ps.sd * (int64_t)sizeof(T);
    const Off voff = (Off)(((int64_t)u * ps.su + (int64_t)v * ps.sv - base0 + (int64_t)k0 * ps.sd) * (int64_t)sizeof(T));
    const int nval = min(NW, ps.nlines - first);   // real lines of this wave
    const int dqN = 64 / N, drN = 64 - dqN * N;    // x lines: walk over N columns
    constexpr int BATCH = 8;

    // ---- partition rows and halo into registers
    T f[W];
    if (xdir) {
        const int e = periodic ? 0 : min(ps.ng, HB + 1);
        const int Tn = N + 2 * e, tp = Tn | 1;
        const int total = nval * Tn;
        const int dq = 64 / Tn, dr = 64 - dq * Tn;
        RowWalk w(lane, Tn, first, -e, ps);
        const T *src = in + fbase;
        for (int e0 = lane; e0 < total; e0 += 64 * BATCH) {
            T val[BATCH];
            int at[BATCH];
#pragma unroll
            for (int b = 0; b < BATCH; ++b) {
                at[b] = -1;
                val[b] = T(0);
                if (e0 + 64 * b < total) {
                    at[b] = w.r * tp + w.j;
                    val[b] = src[w.off];
                }
                w.next(Tn, dq, dr, ps);
            }
#pragma unroll
            for (int b = 0; b < BATCH; ++b)
                if (at[b] >= 0) tile[at[b]] = val[b];
        }
        wave_sync();
        const T *row = tile + l * tp + k0;
        const int ilo = HB + 1 - e, ihi = nlast + e + HB + 1;
#pragma unroll
        for (int i = 0; i < W; ++i) {
            f[i] = T(0);
            if (i < Lr + 2 * HB + 2) {
                if (periodic) {
                    int j = k0 - HB - 1 + i;
                    while (j < 0) j += N;
                    while (j >= N) j -= N;
                    f[i] = tile[l * tp + j];
                } else if (i < ilo || i >= ihi) {
                    const int j = k0 - HB - 1 + i;
                    if (j >= -e && j < N + e) f[i] = row[i - ilo];
                } else {
                    f[i] = row[i - ilo];
                }
            }
        }
        wave_sync();   // the tile is reused for the velocity and the output
    } else if (periodic) {
        const char *src = (const char *)(in + fbase + base0);
        const Off lo = (Off)(((int64_t)u * ps.su + (int64_t)v * ps.sv - base0) * (int64_t)sizeof(T));
#pragma unroll
        for (int i = 0; i < W; ++i) {
            f[i] = T(0);
            if (i < Lr + 2 * HB + 2) {
                int j = k0 - HB - 1 + i;
                while (j < 0) j += N;
                while (j >= N) j -= N;
                f[i] = *(const T *)(src + (Off)(lo + (Off)j * (Off)sdB));
            }
        }
    } else {
        // nodes outside the stored line (a class wider than the scheme, or the
        // missing rows of the last partition) read as 0
        const char *src = (const char *)(in + fbase + base0) - (HB + 1) * sdB;
        const int ilo = HB + 1 - ps.ng, ihi = nlast + ps.ng + HB + 1;
#pragma unroll
        for (int i = 0; i < W; ++i) {
            f[i] = T(0);
            if (i < Lr + 2 * HB + 2) {
                if (i < ilo || i >= ihi) {
                    const int j = k0 - HB - 1 + i;
                    if (j >= -ps.ng && j < N + ps.ng) f[i] = *(const T *)(src + voff);
                } else {
                    f[i] = *(const T *)(src + voff);
                }
            }
            src += sdB;
        }
    }

    // velocity of x lines: through the tile, read back in partition order below
    const int vp = N | 1;
    T *trow = tile + l * vp + k0;
    if (xdir && mode == 0) {
        const int total = nval * N;
        RowWalk w(lane, N, first, 0, ps);
        const T *src = in + ps.vel_base;
        for (int e0 = lane; e0 < total; e0 += 64 * BATCH) {
            T val[BATCH];
            int at[BATCH];
#pragma unroll
            for (int b = 0; b < BATCH; ++b) {
                at[b] = -1;
                val[b] = T(0);
                if (e0 + 64 * b < total) {
                    at[b] = w.r * vp + w.j;
                    val[b] = src[w.off];
                }
                w.next(N, dqN, drN, ps);
            }
#pragma unroll
            for (int b = 0; b < BATCH; ++b)
                if (at[b] >= 0) tile[at[b]] = val[b];
        }
        wave_sync();
    }

    // scans over a line's partitions of v = (value leaving the partition for a
    // zero entering value): lane p's v becomes the value leaving it for a zero
    // value entering the line; wL = the entering value's weight per partition
    auto scan_up = [&](T vv, T wL) {
        for (int s = 1; s < P; s <<= 1) {
            const T t = __shfl(vv, lane - s * NW);
            if (p >= s) vv += wL * t;
            wL *= wL;
        }
        return vv;
    };
    auto scan_down = [&](T vv, T wL) {
        for (int s = 1; s < P; s <<= 1) {
            const T t = __shfl(vv, lane + s * NW);
            if (p + s < P) vv += wL * t;
            wL *= wL;
        }
        return vv;
    };
    const int lastlane = (Pu - 1) * NW + l;

    // ---- right-hand sides (closure rows where this lane holds them)
    const bool closureL = closed && p == 0;
    const bool closureR = closed && islast;
    T rl[L], rr[L];
    if constexpr (EMB) {
        // W: the compact second derivative (2)P1_M on the same rows, explicit
        // closure rows.  [a2, 1, a2] = (1 + b S-)(1 + b S+) b / a2 on the infinite
        // line, so it is a forward and a backward recurrence over the line
        // with zero right side on the closure rows, and the closure values
        // are met with the two homogeneous solutions (-b)^k, (-b)^(N-1-k).
        const T beta = rec[25], kappa = rec[26];
        const T *pb = rec + kBiasPow2;   // (-beta)^n
        const T *st = rec + kBiasSt2, *sc = rec + kBiasCl2;
        T s[L];
        T e0 = T(0), e1 = T(0);
        {
            T up = T(0), uF = T(0), uN = T(0);
#pragma unroll
            for (int i = 0; i < L; ++i) {
                s[i] = T(0);
                if (i < Lr) {
                    T r = st[5] * f[HB + 1 + i];
#pragma unroll
                    for (int m = 1; m <= (HB < 3 ? HB + 1 : 3); ++m)
                        r += st[5 + m] * (f[HB + 1 + i + m] + f[HB + 1 + i - m]);
                    r *= kappa;
                    constexpr int MC = HB + 1 < 5 ? HB + 1 : 5;
                    if (i == 0 && closed) {
                        T c = T(0);
#pragma unroll
                        for (int m = -MC; m <= MC; ++m) c += sc[5 + m] * f[HB + 1 + i + m];
                        e0 = c;
                        if (p == 0) r = T(0);
                    }
                    if (i >= nlast - 1) {
                        if (i == nlast - 1 && closed) {
                            T c = T(0);
#pragma unroll
                            for (int m = -MC; m <= MC; ++m) c += sc[5 - m] * f[HB + 1 + i + m];
                            e1 = c;
                            if (islast) r = T(0);
                        }
                        if (i > nlast - 1 && islast) r = T(0);
                    }
                    const T uu = r - beta * up;
                    s[i] = uu;
                    up = uu;
                    if (i == Lr - 1) uF = uu;
                    if (i == nlast - 1) uN = uu;
                }
            }
            const T vU = scan_up(uF, pb[Lr]);
            T U = __shfl(vU, lane - NW);
            if (p == 0) U = T(0);
            if (periodic) {
                const T xN = __shfl(uN + pb[nlast] * U, lastlane) * (T)ps.wrap2;
                U += pb[k0] * xN;
            }
#pragma unroll
            for (int i = 0; i < L; ++i)
                if (i < Lr) s[i] += pb[i + 1] * U;
        }
        T sn = T(0), sN = T(0);
#pragma unroll
        for (int i = L - 1; i >= 0; --i)
            if (i < Lr) {
                T x = s[i] - beta * sn;
                if (i >= nlast && islast) x = T(0);
                if (i == nlast - 1) sN = x;
                s[i] = x;
                sn = x;
            }
        const T vS = scan_down(idle ? T(0) : s[0], pb[Lr]);
        T S = __shfl(vS, lane + NW);
        if (p + 1 >= P) S = T(0);
        T K1 = T(0), K2 = T(0);
        if (periodic) {
            const T x0 = __shfl(vS, l) * (T)ps.wrap2;
            S += pb[islast || idle ? 0 : N - k0 - Lr] * x0;
        } else {
            const T d0 = __shfl(e0, l) - __shfl(vS, l);
            const T d1 = __shfl(e1, lastlane) - __shfl(sN, lastlane);
            const T bN = pb[N - 1];
            K1 = (d0 - bN * d1) * (T)ps.det2 * pb[k0];
            K2 = (d1 - bN * d0) * (T)ps.det2;
            if (!islast && !idle) K2 *= pb[N - k0 - Lr];
        }
        // the last partition's rows count from its own end, nlast rows in
        K2 -= beta * S;
        if (islast) K2 *= (T)1 / pb[Lr - nlast];
#pragma unroll
        for (int i = 0; i < L; ++i) {
            rl[i] = rr[i] = T(0);
            if (i < Lr) {
                const T e = (T)ps.w2 * (s[i] + K1 * pb[i] + K2 * pb[Lr - 1 - i]);
                rl[i] = left_interior<T, HB>(q, f + i) + e;
                rr[i] = right_interior<T, HB>(q, f + i) - e;
                if (i == 0 && closed) {
                    const T c = left_closure<T, HB>(q, f + i);
                    if (closureL) rl[i] = c;
                }
                if (i == nlast - 1 && closed) {
                    const T c = right_closure<T, HB>(q, f + i);
                    if (closureR) rr[i] = c;
                }
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < L; ++i) {
            rl[i] = rr[i] = T(0);
            if (i < Lr) {
                rl[i] = left_interior<T, HB>(q, f + i);
                rr[i] = right_interior<T, HB>(q, f + i);
                if (i == 0 && closed) {
                    const T c = left_closure<T, HB>(q, f + i);
                    if (closureL) rl[i] = c;
                }
                if (i == nlast - 1 && closed) {
                    const T c = right_closure<T, HB>(q, f + i);
                    if (closureR) rr[i] = c;
                }
            }
        }
        if (ps.s2_in && !idle) {   // U: the sampled second derivative, on every row
            const T *s2 = in + ps.s2_base + (int64_t)u * ps.s2u + (int64_t)v * ps.s2v + (int64_t)k0 * ps.s2d;
            const T w2 = (T)ps.w2, w2c = (T)ps.w2c;
#pragma unroll
            for (int i = 0; i < L; ++i)
                if (i < Lr && !(i >= nlast && islast)) {
                    const T e = s2[(int64_t)i * ps.s2d];
                    rl[i] += ((closureL && i == 0) ? w2c : w2) * e;
                    rr[i] -= ((closureR && i == nlast - 1) ? w2c : w2) * e;
                }
        }
    }

    // ---- local solves with zero entering values
    T xlF = T(0), xlN = T(0);
    if (left) {
        T xp = T(0);
#pragma unroll
        for (int i = 0; i < L; ++i)
            if (i < Lr) {
                T x = rl[i] - alpha * xp;
                if (i == 0 && closureL) x = (rl[0] - alpha * rl[1]) * q.inv_det;
                rl[i] = x;
                xp = x;
                if (i == Lr - 1) xlF = x;
                if (i == nlast - 1) xlN = x;
            }
    }
    if (right) {
        T xn = T(0);
#pragma unroll
        for (int i = L - 1; i >= 0; --i)
            if (i < Lr) {
                T x = rr[i] - alpha * xn;
                if (i > 0 && i == nlast - 1 && closureR) x = (rr[i] - alpha * rr[i > 0 ? i - 1 : 0]) * q.inv_det;
                if (i >= nlast && islast) x = T(0);
                rr[i] = x;
                xn = x;
            }
    }
    // velocity of y/z lines: requested here so that the loads overlap the scans
    T c[L];
    if (mode == 0) {
        if (xdir) {
#pragma unroll
            for (int i = 0; i < L; ++i) c[i] = (i < Lr) ? trow[i] : T(0);
        } else {
            const char *vl = (const char *)(in + ps.vel_base + base0);
#pragma unroll
            for (int i = 0; i < L; ++i) {
                c[i] = T(0);
                if (i < Lr) {
                    if (i < nlast) c[i] = *(const T *)(vl + voff);
                    else if (!islast) c[i] = *(const T *)(vl + voff);
                }
                vl += sdB;
            }
        }
    }

    // ---- true values entering the partition
    T X = T(0), Y = T(0);
    const int64_t eix = 2 * (ps.ev_base + (int64_t)field * ps.nlines + line);   // this line's end entries
    if (left) {
        X = __shfl(scan_up(xlF, pw[Lr]), lane - NW);
        if (p == 0) X = T(0);
        if (periodic) X += pw[k0] * (__shfl(xlN + pw[nlast] * X, lastlane) * (T)ps.wrap);
        if (iter) X += pw[k0] * ev[eix];
        if (ends && !periodic && active && islast) ends[eix] = xlN + pw[nlast] * X;
    }
    if (right) {
        const T vR = scan_down(idle ? T(0) : rr[0], pw[Lr]);
        Y = __shfl(vR, lane + NW);
        if (p + 1 >= P) Y = T(0);
        const int up = (islast || idle) ? 0 : N - k0 - Lr;   // rows above this partition
        if (periodic) Y += pw[up] * (__shfl(vR, l) * (T)ps.wrap);
        if (iter) Y += pw[up] * ev[eix + 1];
        const int nr0 = Pu == 1 ? nlast : Lr;
        if (ends && !periodic && active && p == 0) ends[eix + 1] = rr[0] + pw[nr0] * Y;
        // the last partition's rows count from its own end, nlast rows in
        if ((periodic || iter) && islast && nlast < Lr && alpha != T(0)) Y *= (T)1 / pw[Lr - nlast];
    }

    // ---- corrected values, combined and stored
    const T hinv = (T)ps.hinv;
    const int64_t obase0 = (int64_t)u0 * ps.osu + (int64_t)v0 * ps.osv;
    const int64_t osdB = (int64_t)ps.osd * (int64_t)sizeof(T);
    char *dst = (char *)(out + ps.out_base + (int64_t)field * ps.out_fstride + obase0);
    const Off ovoff =
        (Off)(((int64_t)u * ps.osu + (int64_t)v * ps.osv - obase0 + (int64_t)k0 * ps.osd) * (int64_t)sizeof(T));
    const bool keep = !idle && (xdir || active);
#pragma unroll
    for (int i = 0; i < L; ++i) {
        if (i < Lr) {
            T val;
            if (mode < 0) {
                val = hinv * (rl[i] + pw[i + 1] * X);
            } else if (mode == 1) {
                val = hinv * (rr[i] + pw[Lr - i] * Y);
            } else if (mode == 2) {
                val = T(0.5) * (hinv * (rl[i] + pw[i + 1] * X) + hinv * (rr[i] + pw[Lr - i] * Y));
            } else {
                const T xL = rl[i] + pw[i + 1] * X;
                const T xR = rr[i] + pw[Lr - i] * Y;
                val = fmin(c[i], (T)0) * (hinv * xR) + fmax(c[i], (T)0) * (hinv * xL);
            }
            if (keep && !(i >= nlast && islast)) {
                if (xdir) trow[i] = val;
                else __builtin_nontemporal_store(val, (T *)(dst + ovoff));
            }
        }
        dst += osdB;
    }
    if (xdir) {   // the rows of consecutive x lines are contiguous in the output
        wave_sync();
        const int total = nval * N;
        T *orow = out + ps.out_base + (int64_t)field * ps.out_fstride + (int64_t)first * N;
        int r = lane / N, j = lane - r * N;
#pragma unroll 4
        for (int e = lane; e < total; e += 64) {
            __builtin_nontemporal_store(tile[r * vp + j], orow + e);
            j += drN;
            r += dqN;
            if (j >= N) {
                j -= N;
                ++r;
            }
        }
    }
}

template <typename T, int HB, bool EMB, typename Off, int L0, int... Ls>
__device__ __forceinline__ void bias_dispatch(int code, const BiasPass &ps, int field, int line0, int lgP, int Lr,
                                              int tilew, const T *coefs, const T *in, T *out, const T *ev, T *ends,
                                              T *smem) {
    if (code == 0) {
        bias_wave<T, HB, EMB, L0, Off>(ps, field, line0, lgP, Lr, tilew, coefs, in, out, ev, ends, smem);
        return;
    }
    if constexpr (sizeof...(Ls) > 0)
        bias_dispatch<T, HB, EMB, Off, Ls...>(code - 1, ps, field, line0, lgP, Lr, tilew, coefs, in, out, ev, ends,
                                              smem);
}

// Work item meta: lgP in bits 0..3, Lr in bits 4..11, index of L in the
// kernel's compiled set in bits 12..15.  tilew: elements of one wave's tile.
template <typename T, int HB, bool EMB, typename Off, int... Ls>
__global__ __launch_bounds__(256) void k_biased_wave(const BiasItem *__restrict__ items,
                                                     const BiasPass *__restrict__ passes,
                                                     const T *__restrict__ coefs, const T *__restrict__ in,
                                                     T *__restrict__ out, const T *__restrict__ ev,
                                                     T *__restrict__ ends, int tilew) {
    extern __shared__ __align__(16) unsigned char smem[];
    const BiasItem item = items[blockIdx.x];
    if (item.pass < 0) return;   // padding of the XCD-interleaved order (whole workgroup)
    bias_dispatch<T, HB, EMB, Off, Ls...>((item.meta >> 12) & 15, passes[item.pass], item.field, item.line0,
                                          item.meta & 15, (item.meta >> 4) & 255, tilew, coefs, in, out, ev, ends,
                                          (T *)smem);
}

template <typename T, int HB>
__global__ __launch_bounds__(256) void k_biased(const BiasItem *__restrict__ items, int nitems,
                                                const BiasPass *__restrict__ passes, const T *__restrict__ coefs,
                                                const T *__restrict__ in, T *__restrict__ out) {
    constexpr int W = 2 * HB + 3;
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int it = blockIdx.x * 4 + wv;
    if (it >= nitems) return;
    const BiasItem item = items[it];
    const BiasPass ps = passes[item.pass];
    const int line = item.line0 + lane;
    if (line >= ps.nlines) return;
    const int u = line % ps.nu, v = line / ps.nu;

    BCoef<T, HB> q;
    {
        const T *rec = coefs + (int64_t)ps.tab * kBiasRec;
        q.alpha = rec[0];
        q.inv_det = rec[24];
#pragma unroll
        for (int m = -HB; m <= HB; ++m) q.a[m + HB] = rec[1 + kBiasHalf + m];
#pragma unroll
        for (int m = -HB; m <= HB + 1; ++m) q.c[m + HB] = rec[12 + kBiasHalf + m];
    }
    const int N = ps.N;
    BLine<T> L{in + ps.in_base + (int64_t)item.field * ps.in_fstride + (int64_t)u * ps.su + (int64_t)v * ps.sv,
               ps.sd, N, ps.ng, ps.periodic};
    const T *vel = (ps.mode == 0) ? in + ps.vel_base + (int64_t)u * ps.su + (int64_t)v * ps.sv : nullptr;
    T *o = out + ps.out_base + (int64_t)item.field * ps.out_fstride + (int64_t)u * ps.osu + (int64_t)v * ps.osv;
    const int64_t osd = ps.osd;
    const T hinv = (T)ps.hinv;
    const T alpha = q.alpha;
    T w[W];
    // U: the second-derivative term at node k, interior rows (e2) and closure row (e2c)
    const T *s2 = ps.s2_in ? in + ps.s2_base + (int64_t)u * ps.s2u + (int64_t)v * ps.s2v : nullptr;
    const T w2 = (T)ps.w2, w2c = (T)ps.w2c;
    auto e2 = [&](int k) -> T { return s2 ? w2 * s2[(int64_t)k * ps.s2d] : T(0); };
    auto e2c = [&](int k) -> T { return s2 ? w2c * s2[(int64_t)k * ps.s2d] : T(0); };

    T xl_wrap = 0, xr_wrap = 0;
    if (ps.periodic) {
#pragma unroll
        for (int i = 0; i < W; ++i) w[i] = L.ld(i - (HB + 1));
        T sl = 0, sr = 0, pw = 1;
        for (int k = 0; k < N; ++k) {
            if (ps.mode <= 0 || ps.mode == 2) sl = sl * (-alpha) + (left_interior<T, HB>(q, w) + e2(k));
            if (ps.mode >= 0) {
                sr += pw * (right_interior<T, HB>(q, w) - e2(k));
                pw *= -alpha;
            }
#pragma unroll
            for (int i = 0; i < W - 1; ++i) w[i] = w[i + 1];
            w[W - 1] = L.ld(k + 1 + HB + 1);
        }
        xl_wrap = sl * (T)ps.wrap;
        xr_wrap = sr * (T)ps.wrap;
    }

    // right-biased sweep, k = N-1 .. 0
    if (ps.mode >= 0) {
        auto emit = [&](int k, T x) {
            T val = hinv * x;
            if (ps.mode == 0) val = fmin(vel[(int64_t)k * ps.sd], (T)0) * val;
            if (ps.mode == 2) val = T(0.5) * val;
            o[(int64_t)k * osd] = val;
        };
#pragma unroll
        for (int i = 0; i < W; ++i) w[i] = L.ld(N - 1 - (HB + 1) + i);
        int k = N - 1;
        T xn = xr_wrap;
        if (!ps.periodic) {
            const T rb = right_closure<T, HB>(q, w) - e2c(N - 1);
#pragma unroll
            for (int i = W - 1; i > 0; --i) w[i] = w[i - 1];
            w[0] = L.ld(N - 2 - (HB + 1));
            const T r = right_interior<T, HB>(q, w) - e2(N - 2);
            const T xe = (rb - alpha * r) * q.inv_det;
            xn = r - alpha * xe;
            emit(N - 1, xe);
            emit(N - 2, xn);
#pragma unroll
            for (int i = W - 1; i > 0; --i) w[i] = w[i - 1];
            w[0] = L.ld(N - 3 - (HB + 1));
            k = N - 3;
        }
        for (; k >= 0; --k) {
            const T x = (right_interior<T, HB>(q, w) - e2(k)) - alpha * xn;
            emit(k, x);
            xn = x;
#pragma unroll
            for (int i = W - 1; i > 0; --i) w[i] = w[i - 1];
            w[0] = L.ld(k - 1 - (HB + 1));
        }
    }

    // left-biased sweep, k = 0 .. N-1
    if (ps.mode <= 0 || ps.mode == 2) {
        auto emit = [&](int k, T x) {
            T val = hinv * x;
            if (ps.mode == 0) val = o[(int64_t)k * osd] + fmax(vel[(int64_t)k * ps.sd], (T)0) * val;
            if (ps.mode == 2) val = o[(int64_t)k * osd] + T(0.5) * val;
            o[(int64_t)k * osd] = val;
        };
#pragma unroll
        for (int i = 0; i < W; ++i) w[i] = L.ld(i - (HB + 1));
        int k = 0;
        T xp = xl_wrap;
        if (!ps.periodic) {
            const T rb = left_closure<T, HB>(q, w) + e2c(0);
#pragma unroll
            for (int i = 0; i < W - 1; ++i) w[i] = w[i + 1];
            w[W - 1] = L.ld(1 + HB + 1);
            const T r = left_interior<T, HB>(q, w) + e2(1);
            const T x0 = (rb - alpha * r) * q.inv_det;
            xp = r - alpha * x0;
            emit(0, x0);
            emit(1, xp);
#pragma unroll
            for (int i = 0; i < W - 1; ++i) w[i] = w[i + 1];
            w[W - 1] = L.ld(2 + HB + 1);
            k = 2;
        }
        for (; k < N; ++k) {
            const T x = (left_interior<T, HB>(q, w) + e2(k)) - alpha * xp;
            emit(k, x);
            xp = x;
#pragma unroll
            for (int i = 0; i < W - 1; ++i) w[i] = w[i + 1];
            w[W - 1] = L.ld(k + 1 + HB + 1);
        }
    }
}

template <typename T>
const void *sweep_fn(int hb) {
    switch (hb) {
        case 2: return (const void *)k_biased<T, 2>;
        case 3: return (const void *)k_biased<T, 3>;
        case 4: return (const void *)k_biased<T, 4>;
        case 5: return (const void *)k_biased<T, 5>;
        default: return nullptr;
    }
}

// The wave kernel's instances: partitions of up to 8 or 12 rows (set 0), of up
// to 16 (set 1); with or without an embedded second derivative; 64-bit offsets
// for fields of 4 GiB and more.
template <typename T, int HB>
const void *wave_fn_hb(int set, int emb, int big) {
    if (big) {
        if (set) return emb ? (const void *)k_biased_wave<T, HB, true, uint64_t, 16> : (const void *)k_biased_wave<T, HB, false, uint64_t, 16>;
        return emb ? (const void *)k_biased_wave<T, HB, true, uint64_t, 8, 12> : (const void *)k_biased_wave<T, HB, false, uint64_t, 8, 12>;
    }
    if (set) return emb ? (const void *)k_biased_wave<T, HB, true, uint32_t, 16> : (const void *)k_biased_wave<T, HB, false, uint32_t, 16>;
    return emb ? (const void *)k_biased_wave<T, HB, true, uint32_t, 8, 12> : (const void *)k_biased_wave<T, HB, false, uint32_t, 8, 12>;
}

template <typename T>
const void *wave_fn(int hb, int set, int emb, int big) {
    switch (hb) {
        case 2: return wave_fn_hb<T, 2>(set, emb, big);
        case 3: return wave_fn_hb<T, 3>(set, emb, big);
        case 4: return wave_fn_hb<T, 4>(set, emb, big);
        case 5: return wave_fn_hb<T, 5>(set, emb, big);
        default: return nullptr;
    }
}

}  // namespace

bool biased_supported(int hb) { return hb >= 2 && hb <= 5; }

// The fewest partitions of at most 12 rows (16 on lines of more than 192
// nodes), rows spread evenly, the last partition keeping at least two (its
// closure rows are solved together): fewer partitions keep the stencil halo's
// share of the loads down, and 12 rows of a pair of biases are what fits half
// of a wave's registers.  y and z lines stop at 16 partitions: with fewer than
// 4 lines per wave their accesses cover less than 32 contiguous bytes, and the
// sweep kernel, 64 lines per wave, is the better one.
bool bias_split(int N, int dir, BiasSplit &s) {
    if (N < 2) return false;
    for (int lg = 0; lg <= (dir == 0 ? 6 : 4); ++lg) {
        const int cap = (lg == 4 && N > 192) || lg > 4 ? 16 : 12;
        for (int Lr = std::max(2, (N + (1 << lg) - 1) >> lg); Lr <= cap; ++Lr) {
            const int Pu = (N + Lr - 1) / Lr;
            if (N - (Pu - 1) * Lr < 2) continue;
            s.lgP = lg;
            s.Lr = Lr;
            s.set = Lr > 12;
            s.code = s.set ? 0 : Lr > 8;
            return true;
        }
    }
    return false;
}

int bias_tile_elems(const BiasSplit &s, int dir, int hb, int ng, int periodic, int N) {
    if (dir != 0) return 0;
    const int e = periodic ? 0 : std::min(ng, hb + 1);
    return (64 >> s.lgP) * ((N + 2 * e) | 1);
}

// End values of the next iterate: for every biased pass (rec = ev base of
// the pass, of its left neighbour along the lines, of its right neighbour,
// entries), entry e takes the left neighbour's left-biased last value and the
// right neighbour's right-biased first value of the same field and line.
template <typename T>
__global__ void k_bias_gather(const int64_t *__restrict__ recs, const T *__restrict__ ends, T *__restrict__ ev) {
    const int64_t *r = recs + 4 * blockIdx.y;
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= r[3]) return;
    ev[2 * (r[0] + e)] = ends[2 * (r[1] + e)];
    ev[2 * (r[0] + e) + 1] = ends[2 * (r[2] + e) + 1];
}

hipError_t launch_bias_gather(int f32, int npass, int64_t max_entries, const int64_t *recs, const void *ends, void *ev,
                              hipStream_t st) {
    if (npass == 0 || max_entries == 0) return hipSuccess;
    const dim3 grid((unsigned)((max_entries + 255) / 256), (unsigned)npass);
    if (f32)
        hipLaunchKernelGGL(k_bias_gather<float>, grid, dim3(256), 0, st, recs, (const float *)ends, (float *)ev);
    else
        hipLaunchKernelGGL(k_bias_gather<double>, grid, dim3(256), 0, st, recs, (const double *)ends, (double *)ev);
    return hipGetLastError();
}

hipError_t launch_biased(int f32, const BiasLaunch &g, const BiasItem *items, const BiasPass *passes,
                         const void *coefs, const void *in, void *out, const void *ev, void *ends, hipStream_t st) {
    if (g.nitems <= 0) return hipSuccess;
    if (g.sweep) {
        const int grid = (g.nitems + 3) / 4;
        const void *fn = f32 ? sweep_fn<float>(g.hb) : sweep_fn<double>(g.hb);
        if (!fn) return hipErrorInvalidValue;
        if (f32)
            hipLaunchKernelGGL(((void (*)(const BiasItem *, int, const BiasPass *, const float *, const float *,
                                          float *))fn),
                               dim3(grid), dim3(256), 0, st, items, g.nitems, passes, (const float *)coefs,
                               (const float *)in, (float *)out);
        else
            hipLaunchKernelGGL(((void (*)(const BiasItem *, int, const BiasPass *, const double *, const double *,
                                          double *))fn),
                               dim3(grid), dim3(256), 0, st, items, g.nitems, passes, (const double *)coefs,
                               (const double *)in, (double *)out);
        return hipGetLastError();
    }
    const void *fn = f32 ? wave_fn<float>(g.hb, g.set, g.emb, g.big) : wave_fn<double>(g.hb, g.set, g.emb, g.big);
    if (!fn) return hipErrorInvalidValue;
    const size_t lds = (size_t)4 * g.tilew * (f32 ? 4 : 8);
    if (f32)
        hipLaunchKernelGGL(((void (*)(const BiasItem *, const BiasPass *, const float *, const float *, float *,
                                      const float *, float *, int))fn),
                           dim3(g.nitems), dim3(256), lds, st, items, passes, (const float *)coefs, (const float *)in,
                           (float *)out, (const float *)ev, (float *)ends, g.tilew);
    else
        hipLaunchKernelGGL(((void (*)(const BiasItem *, const BiasPass *, const double *, const double *, double *,
                                      const double *, double *, int))fn),
                           dim3(g.nitems), dim3(256), lds, st, items, passes, (const double *)coefs,
                           (const double *)in, (double *)out, (const double *)ev, (double *)ends, g.tilew);
    return hipGetLastError();
}

}  // namespace cfd
