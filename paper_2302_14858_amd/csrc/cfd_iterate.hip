// Hybrid iteration of the block closures (arXiv 2302.14858,
// Sec. ssec:domdec_iter, Eq. iter_center_P and its matrix form Eq. iter_scheme).
//
// On a periodic lattice of blocks, iterate i > 0 of a tridiagonal scheme solves
// each block line with the derivative two nodes past either end fixed to the
// neighbouring block's iterate i - 1 there.  Written on the block's own nodes
// (the host's make_iterated), that is a closure system with implicit closure
// rows whose right side carries gamma times each end value, so
//   x^[i] = xf + e-^[i-1] g- + e+^[i-1] g+,
// with xf the solution for zero end values and g-, g+ fixed influence vectors.
// Only two values per line pass between the blocks: the iterate at nodes c - 1
// and N - c (c = 2), which the neighbours read as their end values.  The
// device work per apply:
//   1. k_end_values: per line, the iterate-0 values at those nodes (the block
//      closure of Eq. sch_cent_om) and the xf values there, as dot products of
//      the line with rows of h^-d D_L^-1 D_R built once per plan
//      (k_end_weights, FP64);
//   2. k_iter_ends: the end-node values of the next iterate from the
//      neighbours' current ones (no pass over the fields);
//   3. the line kernel of the iterated system (EXT class), which adds
//      e- g- + e+ g+ to its solution.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "cfd_internal.h"

namespace cfd {

// One weight table: both systems of one (scheme, N), FP64.
struct EndWeightSpec {
    int N, c, d;                 // line length, end-node offset, derivative degree
    double alpha;                // interior alpha^(d)_{+-1}
    double a[2 * kMaxHalf + 1];  // interior stencil
    double cl[2 * kMaxHalf + 1]; // block-closure stencil of row k*_- (identity row of D_L)
    double ce[2 * kMaxHalf + 1]; // iterated closure stencil of row k*_-
    double cl_d0, cl_up;         // iterated closure row of D_L
    int64_t off;                 // output: 4 x (N + 2 kMaxHalf) doubles
};

// Row `row` of D_R (stencil centred at node row, over nodes -R .. N+R-1) of
// system ext (0: block closure, 1: iterated closure), accumulated with weight z.
__device__ inline void add_dr_row(const EndWeightSpec &s, int ext, int row, double z, double *w) {
    constexpr int R = kMaxHalf;
    const double sgn = (s.d % 2) ? -1.0 : 1.0;
    const double *st;
    bool mirror = false;
    if (row == 0) st = ext ? s.ce : s.cl;
    else if (row == s.N - 1) { st = ext ? s.ce : s.cl; mirror = true; }
    else st = s.a;
    for (int m = -R; m <= R; ++m) {
        const double v = mirror ? sgn * st[R - m] : st[R + m];
        if (v != 0.0) w[row + m + R] += z * v;
    }
}

// Thread (table, q): q = 0, 1 block closure at rows c - 1, N - c; q = 2, 3 the
// iterated system at the same rows.  Row j of D_L^-1 D_R is z^T D_R with
// D_L^T z = e_j, a tridiagonal solve without pivoting.
__global__ void k_end_weights(int ntab, const EndWeightSpec *__restrict__ specs, double *__restrict__ data,
                              double *__restrict__ scratch, int stride) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 4 * ntab) return;
    const EndWeightSpec s = specs[t / 4];
    const int q = t % 4;
    const int ext = q >= 2;
    const int N = s.N;
    const int j = (q % 2) ? N - s.c : s.c - 1;
    double *cp = scratch + (int64_t)t * 2 * stride;   // stride >= every table's N
    double *z = cp + N;
    // D_L rows: (lo, di, up)
    auto lo = [&](int r) -> double {
        if (r == 0) return 0.0;
        if (r == N - 1) return ext ? s.cl_up : 0.0;
        return s.alpha;
    };
    auto up = [&](int r) -> double {
        if (r == N - 1) return 0.0;
        if (r == 0) return ext ? s.cl_up : 0.0;
        return s.alpha;
    };
    auto di = [&](int r) -> double { return (r == 0 || r == N - 1) ? (ext ? s.cl_d0 : 1.0) : 1.0; };
    // D_L^T: sub-diagonal up(r-1), diagonal di(r), super-diagonal lo(r+1)
    for (int r = 0; r < N; ++r) {
        const double sub = r > 0 ? up(r - 1) : 0.0;
        const double sup = r + 1 < N ? lo(r + 1) : 0.0;
        const double rhs = r == j ? 1.0 : 0.0;
        const double m = di(r) - (r > 0 ? sub * cp[r - 1] : 0.0);
        cp[r] = sup / m;
        z[r] = (rhs - (r > 0 ? sub * z[r - 1] : 0.0)) / m;
    }
    for (int r = N - 2; r >= 0; --r) z[r] -= cp[r] * z[r + 1];
    double *w = data + s.off + (int64_t)q * (N + 2 * kMaxHalf);
    for (int k = 0; k < N + 2 * kMaxHalf; ++k) w[k] = 0.0;
    for (int r = 0; r < N; ++r) add_dr_row(s, ext, r, z[r], w);
}

// One (pass, operator) of an iterated plan, with its lines' end values at
// units ubase .. ubase + nunits - 1 (unit = field * nlines + line, two values
// each: the left and right end-node values, or end values).
struct IterOp {
    int pass, o;
    int nbr_m, nbr_p;            // the same pass and operator on the neighbouring blocks
    int64_t ubase;
    int nunits;
    int N, c, Npad;
    int64_t wofs;                // end weights (4 x (N + 2 kMaxHalf) doubles)
    int64_t gofs;                // influence vectors g-, g+ in the FP64 tables ([2][Npad])
    double hinv;
};

// End values are kept where they are read: slot 2 e of a line's entry e holds
// its left end value (the left neighbour's value at N - c) and slot 2 e + 1 its
// right one (the right neighbour's at c - 1), so a line's own end-node values
// go to its neighbours' slots.
template <typename T>
__device__ __forceinline__ void put_ends(const IterOp *ops, const IterOp &op, int u, T *ev, T left, T right) {
    ev[2 * (ops[op.nbr_m].ubase + u) + 1] = left;
    ev[2 * (ops[op.nbr_p].ubase + u)] = right;
}

// Per line: the iterate-0 end-node values into ev0 and the xf values there into
// endsf.  A workgroup takes 64 lines (lane = line) and cuts their nodes into
// four runs, one per wave, so that the weights are wave-uniform (scalar loads)
// and the loads of a line are in flight from four waves; the partial sums meet
// in LDS.  x lines are staged through an LDS tile with contiguous loads (64
// blocks of 32^3, 5 fields, FP64, three directions: 52 us; one lane per
// line with the x lines read in place, 124 us).
template <typename T>
__global__ void __launch_bounds__(256)
k_end_values(const IterOp *__restrict__ ops, const PassDesc *__restrict__ passes, const double *__restrict__ weights,
             const T *__restrict__ in, T *__restrict__ ev0, T *__restrict__ endsf) {
    extern __shared__ __align__(16) unsigned char smem[];
    const IterOp &op = ops[blockIdx.y];
    const int u0 = blockIdx.x * 64;
    if (u0 >= op.nunits) return;   // whole workgroup
    const PassDesc &pd = passes[op.pass];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nlines = pd.nlines, N = op.N;
    constexpr int R = kMaxHalf;
    const int e = min(R, pd.ng);       // stored nodes -e .. N + e - 1; weights beyond are zero
    const int Tn = N + 2 * e, tp = Tn | 1;
    const int q = (Tn + 3) / 4;
    const int j0 = wv * q, j1 = min(j0 + q, Tn);
    auto line_of = [&](int u) -> int64_t {   // offset of node -e of unit u's line
        const int f = u / nlines, line = u - f * nlines;
        const int lv = line / pd.nu, lu = line - lv * pd.nu;
        return pd.in_base + (int64_t)(pd.field0 + f) * pd.in_fstride + (int64_t)lv * pd.sv + (int64_t)lu * pd.su -
               (int64_t)e * pd.sd;
    };
    const int u = min(u0 + lane, op.nunits - 1);
    const int64_t mine = line_of(u);
    T *part = (T *)smem;               // [4 waves][4 sums][64 lanes]
    const double *w = weights + op.wofs + (R - e);
    const int W = N + 2 * R;
    T s0 = 0, s1 = 0, s2 = 0, s3 = 0;
    auto add = [&](int j, T v) {
        s0 += (T)w[j] * v;
        s1 += (T)w[W + j] * v;
        s2 += (T)w[2 * W + j] * v;
        s3 += (T)w[3 * W + j] * v;
    };
    constexpr int B = 8;
    if (pd.sd == 1) {
        T *tile = part + 16 * 64;
        int64_t *rows = (int64_t *)part;   // line offsets, until the partial sums
        if (wv == 0) rows[lane] = mine;
        __syncthreads();
        const int total = 64 * Tn;
        int r = threadIdx.x / Tn, j = threadIdx.x - r * Tn;
        const int dr = 256 / Tn, dj = 256 - dr * Tn;
        for (int k0 = threadIdx.x; k0 < total; k0 += 256 * B) {
            T v[B];
            int at[B];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                at[b] = -1;
                if (k0 + 256 * b < total) {
                    at[b] = r * tp + j;
                    v[b] = in[rows[r] + j];
                    r += dr;
                    j += dj;
                    if (j >= Tn) {
                        j -= Tn;
                        ++r;
                    }
                }
            }
#pragma unroll
            for (int b = 0; b < B; ++b)
                if (at[b] >= 0) tile[at[b]] = v[b];
        }
        __syncthreads();
        for (int jj = j0; jj < j1; ++jj) add(jj, tile[lane * tp + jj]);
    } else {
        const T *src = in + mine;
        int jj = j0;
        for (; jj + B <= j1; jj += B) {
            T v[B];
#pragma unroll
            for (int b = 0; b < B; ++b) v[b] = src[(int64_t)(jj + b) * pd.sd];
#pragma unroll
            for (int b = 0; b < B; ++b) add(jj + b, v[b]);
        }
        for (; jj < j1; ++jj) add(jj, src[(int64_t)jj * pd.sd]);
    }
    part[(wv * 4 + 0) * 64 + lane] = s0;
    part[(wv * 4 + 1) * 64 + lane] = s1;
    part[(wv * 4 + 2) * 64 + lane] = s2;
    part[(wv * 4 + 3) * 64 + lane] = s3;
    __syncthreads();
    if (wv != 0 || u0 + lane >= op.nunits) return;
    T s[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        s[k] = (part[k * 64 + lane] + part[(4 + k) * 64 + lane]) + (part[(8 + k) * 64 + lane] + part[(12 + k) * 64 + lane]);
    const T h = (T)op.hinv;
    put_ends(ops, op, u, ev0, h * s[0], h * s[1]);
    const int64_t en = 2 * (op.ubase + u);
    endsf[en] = h * s[2];
    endsf[en + 1] = h * s[3];
}

// One exchange step: every line's end-node values of the next iterate from its
// end values (prev), into its neighbours' slots of next.
template <typename T>
__global__ void k_iter_ends(const IterOp *__restrict__ ops, const double *__restrict__ tabs64,
                            const T *__restrict__ endsf, const T *__restrict__ prev, T *__restrict__ next) {
    const IterOp op = ops[blockIdx.y];
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= op.nunits) return;
    const int64_t e = 2 * (op.ubase + u);
    const T em = prev[e], ep = prev[e + 1];
    const double *gm = tabs64 + op.gofs, *gp = gm + op.Npad;
    const int jl = op.c - 1, jr = op.N - op.c;
    put_ends(ops, op, u, next, endsf[e] + (T)gm[jl] * em + (T)gp[jl] * ep,
             endsf[e + 1] + (T)gm[jr] * em + (T)gp[jr] * ep);
}

size_t end_weight_spec_size() { return sizeof(EndWeightSpec); }
size_t iter_op_size() { return sizeof(IterOp); }

void fill_end_weight_spec(void *dst, int N, int c, const Scheme &blk, const Scheme &it, int64_t off) {
    EndWeightSpec s;
    s.N = N;
    s.c = c;
    s.d = blk.d;
    s.alpha = blk.lhs[kMaxNL + 1];
    for (int m = 0; m < 2 * kMaxHalf + 1; ++m) {
        s.a[m] = blk.rhs[m];
        s.cl[m] = blk.cl[0][m];
        s.ce[m] = it.cl[0][m];
    }
    s.cl_d0 = it.cl_d0;
    s.cl_up = it.cl_up;
    s.off = off;
    *reinterpret_cast<EndWeightSpec *>(dst) = s;
}

void fill_iter_op(void *dst, int pass, int o, int nbr_m, int nbr_p, int64_t ubase, int nunits, int N, int c, int Npad,
                  int64_t wofs, int64_t gofs, double hinv) {
    IterOp r;
    r.pass = pass;
    r.o = o;
    r.nbr_m = nbr_m;
    r.nbr_p = nbr_p;
    r.ubase = ubase;
    r.nunits = nunits;
    r.N = N;
    r.c = c;
    r.Npad = Npad;
    r.wofs = wofs;
    r.gofs = gofs;
    r.hinv = hinv;
    *reinterpret_cast<IterOp *>(dst) = r;
}

hipError_t launch_end_weights(int ntab, const void *specs, double *data, double *scratch, int stride, hipStream_t st) {
    hipLaunchKernelGGL(k_end_weights, dim3((4 * ntab + 63) / 64), dim3(64), 0, st, ntab,
                       (const EndWeightSpec *)specs, data, scratch, stride);
    return hipGetLastError();
}

size_t end_values_lds(int f32, int max_N) {
    return (size_t)64 * (16 + ((max_N + 2 * kMaxHalf) | 1)) * (f32 ? 4 : 8);
}

hipError_t launch_end_values(int f32, int nops, int max_units, int max_N, const void *ops, const PassDesc *passes,
                             const double *weights, const void *in, void *ev0, void *endsf, hipStream_t st) {
    const dim3 grid((max_units + 63) / 64, nops);
    const size_t lds = end_values_lds(f32, max_N);
    if (f32)
        hipLaunchKernelGGL(k_end_values<float>, grid, dim3(256), lds, st, (const IterOp *)ops, passes, weights,
                           (const float *)in, (float *)ev0, (float *)endsf);
    else
        hipLaunchKernelGGL(k_end_values<double>, grid, dim3(256), lds, st, (const IterOp *)ops, passes, weights,
                           (const double *)in, (double *)ev0, (double *)endsf);
    return hipGetLastError();
}

hipError_t launch_iter_ends(int f32, int nops, int max_units, const void *ops, const double *tabs64, const void *endsf,
                            const void *prev, void *next, hipStream_t st) {
    const dim3 grid((max_units + 255) / 256, nops);
    if (f32)
        hipLaunchKernelGGL(k_iter_ends<float>, grid, dim3(256), 0, st, (const IterOp *)ops, tabs64,
                           (const float *)endsf, (const float *)prev, (float *)next);
    else
        hipLaunchKernelGGL(k_iter_ends<double>, grid, dim3(256), 0, st, (const IterOp *)ops, tabs64,
                           (const double *)endsf, (const double *)prev, (double *)next);
    return hipGetLastError();
}

}  // namespace cfd
