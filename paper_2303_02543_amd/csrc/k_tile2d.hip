// 2D Jacobi pass for grids too small to fill the GPU with marching strips: a
// workgroup holds a tile of the grid in registers and runs all sweeps of the
// pass on it.
//
// The update is the 5-point Jacobi step of the proxy application in Section
// 4.3 of the paper, s = (W + E) + (S + N); u' = (s + b) * 1/4, with no FMA
// contraction, so the pass gives the same bits as every other schedule.
//
// A workgroup of 16 waves holds a tile of 64 V columns by 16 RY rows; a lane
// holds V columns of RY consecutive rows, and the source there, from the first
// sweep to the last.  x neighbours come from DPP wave shifts, y neighbours
// from the lane's own rows and, at a wave's first and last row, from the
// neighbouring waves' rows in LDS (two buffers alternate by sweep, one barrier
// per sweep).  Cells are read from whichever block owns them, once.  Every
// sweep invalidates one more cell on each side of the tile that does not border
// the Dirichlet ring, so a pass of t sweeps outputs the tile less t rows and
// (t rounded up to V) columns there; at the ring the tile needs no halo: the
// ring column beside it rides in a register, the ring row in the LDS slot of
// the wave that would lie beyond.
//
// Why: the marching pass (k_march2d) runs a tile row by row, 2 t + rows steps
// of ~0.5 us each in series, whatever the grid's size; a tile in registers
// takes ~0.2 us per sweep.  Its redundancy is higher (a 128 x 64 tile outputs
// 104 x 40 after 12 sweeps) and its loads are not overlapped with arithmetic,
// so grids that fill the GPU with strips march (tile2d_plan holds the rule).
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "jacobi_internal.h"
#include "kernels.h"

namespace jac {

constexpr int kT2Waves = 16;
enum { T2_LAPLACE = 0, T2_POISSON = 1, T2_ADJOINT = 2 };

template <typename R, int V>
struct alignas(V * sizeof(R)) Cells {
    R v[V];
};

struct T2Args {
    int t, nstrips, ngrp, nitems, acols;
    int nt;  // store the outputs with the non-temporal hint
};

template <typename R, int V, int RY>
struct T2Lane {
    int nxr;      // interior columns from the lane's first on
    int nyr;      // interior rows from the wave's first on
    int o0, o1;   // rows [o0, o1) of the wave are outputs
    bool out;     // the lane's columns are outputs (those < nxr)
    int lane, wv;
    R e[RY];      // EDGE: ring cell beside the tile (lanes 0, 63)
    double acc;   // residual partial
};

template <typename R, int V>
using T2Sh = Cells<R, V> (*)[kT2Waves + 2][2][64];

// The rows just above and below the wave's own, through buffer `par` of the
// LDS rows.
template <typename R, int V, int RY>
__device__ __forceinline__ void t2_rows_of(const R (&cur)[RY][V], const T2Lane<R, V, RY> &L,
                                           T2Sh<R, V> sh, int par, Cells<R, V> &so,
                                           Cells<R, V> &no) {
    Cells<R, V> lo, hi;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        lo.v[v] = cur[0][v];
        hi.v[v] = cur[RY - 1][v];
    }
    sh[par][L.wv + 1][0][L.lane] = lo;
    sh[par][L.wv + 1][1][L.lane] = hi;
    __syncthreads();
    so = sh[par][L.wv][1][L.lane];
    no = sh[par][L.wv + 2][0][L.lane];
}

// Residual partial of the pass's input, FP64 from widened values.
template <typename R, int V, int RY, int MODE, bool EDGE>
__device__ __forceinline__ void t2_residual(const R (&cur)[RY][V], const R (&b)[RY][V],
                                            T2Lane<R, V, RY> &L, T2Sh<R, V> sh) {
    Cells<R, V> so, no;
    t2_rows_of<R, V, RY>(cur, L, sh, 1, so, no);
#pragma unroll
    for (int j = 0; j < RY; ++j) {
        const R eo = EDGE ? L.e[j] : (R)0;
        const R left = shift_up(eo, cur[j][V - 1]);
        const R right = shift_down(eo, cur[j][0]);
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const double Wd = v > 0 ? cur[j][v - 1] : left;
            const double Ed = v < V - 1 ? cur[j][v + 1] : right;
            const double Sd = j > 0 ? cur[j - 1][v] : so.v[v];
            const double Nd = j < RY - 1 ? cur[j + 1][v] : no.v[v];
            const double sd = (Wd + Ed) + (Sd + Nd);
            const double bd = MODE == T2_POISSON ? (double)b[j][v] : 0.0;
            const double r = bd - (4.0 * (double)cur[j][v] - sd);
            const bool mine = L.out && j >= L.o0 && j < L.o1 && (!EDGE || v < L.nxr);
            L.acc += mine ? r * r : 0.0;
        }
    }
}

// One sweep from cur to nxt; buffer `par` of the LDS rows.
template <typename R, int V, int RY, int MODE, bool EDGE>
__device__ __forceinline__ void t2_sweep(const R (&cur)[RY][V], R (&nxt)[RY][V],
                                         const R (&b)[RY][V], double (&ga)[RY][V],
                                         T2Lane<R, V, RY> &L, T2Sh<R, V> sh, int par) {
    Cells<R, V> so, no;
    t2_rows_of<R, V, RY>(cur, L, sh, par, so, no);
    const R w = (R)0.25;
#pragma unroll
    for (int jj = 0; jj < RY; ++jj) {
        // the rows that need no LDS row first
        const int j = RY < 3 ? jj : jj < RY - 2 ? jj + 1 : jj == RY - 2 ? 0 : RY - 1;
        const R eo = EDGE ? L.e[j] : (R)0;
        const R left = shift_up(eo, cur[j][V - 1]);
        const R right = shift_down(eo, cur[j][0]);
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const R Wv = v > 0 ? cur[j][v - 1] : left;
            const R Ev = v < V - 1 ? cur[j][v + 1] : right;
            const R Sv = j > 0 ? cur[j - 1][v] : so.v[v];
            const R Nv = j < RY - 1 ? cur[j + 1][v] : no.v[v];
            const R s = (Wv + Ev) + (Sv + Nv);
            R o = MODE == T2_POISSON ? (s + b[j][v]) * w : s * w;
            // adjoint: the level swept from is the next term of the sum
            if constexpr (MODE == T2_ADJOINT) ga[j][v] += (double)(w * cur[j][v]);
            // ring cells and cells beyond the ring keep their values
            if constexpr (EDGE) o = (v < L.nxr && j < L.nyr) ? o : cur[j][v];
            nxt[j][v] = o;
        }
    }
}

// Element offsets of a wave's rows in the state and source buffers (uniform:
// one division for the first row, the others counted on).
template <int RY>
struct T2Rows {
    int64_t su[RY], sb[RY];
};
template <int RY>
__device__ __forceinline__ T2Rows<RY> t2_rows(const Geom &g, int y) {
    T2Rows<RY> r;
    const int ny = g.n[1];
    int by, ly;
    owner(y > ny ? ny : y, g.e[1], g.nb[1], by, ly);
#pragma unroll
    for (int j = 0; j < RY; ++j) {
        r.su[j] = (int64_t)by * g.nb[0] * g.bstride + (int64_t)(ly + 1) * g.pitch;
        r.sb[j] = y + j < ny ? (int64_t)by * g.nb[0] * g.sstride + (int64_t)ly * g.e[0] : 0;
        if (y + j < ny) {  // rows beyond the ring stay on its row
            ++ly;
            if (ly >= g.e[1] && by < g.nb[1] - 1) {
                ++by;
                ly = 0;
            }
        }
    }
    return r;
}

template <typename R, int V, int RY>
__device__ __forceinline__ void t2_store(R *__restrict__ uout, const R (&val)[RY][V],
                                         const T2Lane<R, V, RY> &L, const T2Rows<RY> &rows,
                                         uint32_t col, bool nt) {
    if (!uout) return;
#pragma unroll
    for (int j = 0; j < RY; ++j) {
        if (j < L.o0 || j >= L.o1) continue;
        R *d = uout + rows.su[j];
        if (L.out && L.nxr >= V) {
            Cells<R, V> t;
#pragma unroll
            for (int v = 0; v < V; ++v) t.v[v] = val[j][v];
            if (nt)
                store_nt(&at_mut<Cells<R, V>>(d, col), t);
            else
                at_mut<Cells<R, V>>(d, col) = t;
        } else if (L.out) {
#pragma unroll
            for (int v = 0; v < V; ++v)
                if (v < L.nxr) at_mut<R>(d, col + v * (uint32_t)sizeof(R)) = val[j][v];
        }
    }
}

template <typename R, int V, int RY, int MODE, bool EDGE, bool RES>
__device__ __forceinline__ void t2_body(const Geom &g, const R *__restrict__ uin,
                                        R *__restrict__ uout, const R *__restrict__ bsrc,
                                        double *__restrict__ gacc, T2Lane<R, V, RY> &L,
                                        T2Sh<R, V> sh, int t, int a, int c, int y, bool nt) {
    using C = Cells<R, V>;
    const int nx = g.n[0], ny = g.n[1];
    R p[RY][V], q[RY][V], b[RY][V];
    double ga[RY][V];
    // columns and rows beyond the ring are read from in-bounds stand-ins; they
    // only ever feed cells that are kept or not output
    int bx, lx, ex, elx;
    owner(c <= nx ? c : 0, g.e[0], g.nb[0], bx, lx);
    const int xe = L.lane == 0 ? a - 1 : a + 64 * V;
    owner(xe <= nx ? xe : 0, g.e[0], g.nb[0], ex, elx);
    const uint32_t col = (uint32_t)(((int64_t)bx * g.bstride + g.ax + lx) * (int64_t)sizeof(R));
    const uint32_t ecol = (uint32_t)(((int64_t)ex * g.bstride + g.ax + elx) * (int64_t)sizeof(R));
    const uint32_t scol =
        (uint32_t)(((int64_t)bx * g.sstride + (c < nx ? lx : 0)) * (int64_t)sizeof(R));
    const T2Rows<RY> rows = t2_rows<RY>(g, y);
    C t0[RY], t1[RY];
#pragma unroll
    for (int j = 0; j < RY; ++j) {
        t0[j] = at<C>(uin + rows.su[j], col);
        L.e[j] = EDGE ? at<R>(uin + rows.su[j], ecol) : (R)0;
        if constexpr (MODE == T2_POISSON) t1[j] = at<C>(bsrc + rows.sb[j], scol);
    }
#pragma unroll
    for (int j = 0; j < RY; ++j)
#pragma unroll
        for (int v = 0; v < V; ++v) {
            p[j][v] = t0[j].v[v];
            b[j][v] = MODE == T2_POISSON ? t1[j].v[v] : (R)0;
            ga[j][v] = 0.0;
        }
    // the accumulator of the lane's output cells: whole chunks where the
    // chunk is interior (the array's rows are 8-byte aligned only)
    struct __attribute__((packed, aligned(8))) Acc {
        double v[V];
    };
    if constexpr (MODE == T2_ADJOINT) {
#pragma unroll
        for (int j = 0; j < RY; ++j) {
            if (!L.out || j < L.o0 || j >= L.o1) continue;
            const double *s = gacc + (int64_t)(y + j) * nx + c;
            if (L.nxr >= V) {
                const Acc x = *reinterpret_cast<const Acc *>(s);
#pragma unroll
                for (int v = 0; v < V; ++v) ga[j][v] = x.v[v];
            } else {
#pragma unroll
                for (int v = 0; v < V; ++v)
                    if (v < L.nxr) ga[j][v] = s[v];
            }
        }
    }
    // the rows just outside the tile: the ring's row where the tile borders
    // it (any values elsewhere), the same for every sweep
    if (L.wv == 0 || L.wv == kT2Waves - 1) {
        const int yo = L.wv == 0 ? y - 1 : y + RY;
        int by, ly;
        owner(yo > ny ? ny : yo, g.e[1], g.nb[1], by, ly);
        const C r = at<C>(uin + (int64_t)by * g.nb[0] * g.bstride + (int64_t)(ly + 1) * g.pitch, col);
        const int slot = L.wv == 0 ? 0 : kT2Waves + 1;
        sh[0][slot][L.wv == 0 ? 1 : 0][L.lane] = r;
        sh[1][slot][L.wv == 0 ? 1 : 0][L.lane] = r;
    }
    if constexpr (RES) {
        t2_residual<R, V, RY, MODE, EDGE>(p, b, L, sh);
        // the sum is taken here: left to itself the compiler moves it to its
        // use at the kernel's end, with every row's neighbours held till then
        asm volatile("" : "+v"(L.acc));
    }
    for (int i = 0; i + 1 < t; i += 2) {
        t2_sweep<R, V, RY, MODE, EDGE>(p, q, b, ga, L, sh, 0);
        t2_sweep<R, V, RY, MODE, EDGE>(q, p, b, ga, L, sh, 1);
    }
    if (t & 1) {
        t2_sweep<R, V, RY, MODE, EDGE>(p, q, b, ga, L, sh, 0);
        t2_store<R, V, RY>(uout, q, L, rows, col, nt);
    } else {
        t2_store<R, V, RY>(uout, p, L, rows, col, nt);
    }
    if constexpr (MODE == T2_ADJOINT) {
#pragma unroll
        for (int j = 0; j < RY; ++j) {
            if (!L.out || j < L.o0 || j >= L.o1) continue;
            double *d = gacc + (int64_t)(y + j) * nx + c;
            if (L.nxr >= V) {
                Acc x;
#pragma unroll
                for (int v = 0; v < V; ++v) x.v[v] = ga[j][v];
                *reinterpret_cast<Acc *>(d) = x;
            } else {
#pragma unroll
                for (int v = 0; v < V; ++v)
                    if (v < L.nxr) d[v] = ga[j][v];
            }
        }
    }
}

// uout may be NULL (residual only); res (used when RES) receives one residual
// partial per work item; gacc is the FP64 accumulator of the adjoint pass.
template <typename R, int V, int RY, int MODE, bool RES>
__global__ __launch_bounds__(64 * kT2Waves) void k_tile2d(Geom g, const R *__restrict__ uin,
                                                         R *__restrict__ uout,
                                                         const R *__restrict__ bsrc,
                                                         double *__restrict__ res,
                                                         double *__restrict__ gacc, T2Args A) {
    constexpr int W = 64 * V, H = kT2Waves * RY;
    __shared__ Cells<R, V> sh[2][kT2Waves + 2][2][64];
    __shared__ double part[kT2Waves];
    const int item = xcd_logical_block(blockIdx.x, gridDim.x);
    if (item >= A.nitems) return;  // whole workgroup
    const int strip = item % A.nstrips, grp = item / A.nstrips;
    const int nx = g.n[0], ny = g.n[1], t = A.t;
    T2Lane<R, V, RY> L;
    L.wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    L.lane = threadIdx.x & 63;
    const int a = strip * (W - 2 * A.acols), y0 = grp * (H - 2 * t);
    const int c = a + L.lane * V, y = y0 + L.wv * RY;
    L.nxr = nx - c;
    L.nyr = ny - y;
    const int ylo = grp == 0 ? 0 : y0 + t, yhi = grp == A.ngrp - 1 ? ny : y0 + H - t;
    L.o0 = ylo - y;
    L.o1 = yhi - y;
    const int xlo = strip == 0 ? 0 : a + A.acols;
    const int xhi = strip == A.nstrips - 1 ? nx : a + W - A.acols;
    L.out = c >= xlo && c < xhi;
    L.acc = 0.0;
    if (a == 0 || a + W >= nx || y0 + H > ny)
        t2_body<R, V, RY, MODE, true, RES>(g, uin, uout, bsrc, gacc, L, sh, t, a, c, y,
                                          MODE != T2_ADJOINT && A.nt != 0);
    else
        t2_body<R, V, RY, MODE, false, RES>(g, uin, uout, bsrc, gacc, L, sh, t, a, c, y,
                                          MODE != T2_ADJOINT && A.nt != 0);
    if constexpr (RES) {
        const double s = wave_sum(L.acc);
        if (L.lane == 0) part[L.wv] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            double total = part[0];
#pragma unroll
            for (int k = 1; k < kT2Waves; ++k) total += part[k];
            res[item] = total;
        }
    }
}

// ---- host side -------------------------------------------------------------
// The kernels of each type are compiled in an object of their own (this file
// built with JAC_TILE2D_TYPE=float / double); the object built without it
// holds the dispatch and the schedule rule.
template <typename R>
hipError_t t2_launch_r(const Geom &g, const void *uin, void *uout, const void *b, double *res,
                       double *gacc, const Tile2dPlan &pl, hipStream_t st);

// Tile shapes (columns per lane, rows per lane), smallest first.
struct T2Shape {
    int v, ry;
};
template <typename R>
static const T2Shape *t2_shapes(int *n) {
    static const T2Shape s[] = {{1, 2}, {1, 4}, {2, 4}, {2, 8}, {4, 8}};
    *n = sizeof(R) == 4 ? 5 : 4;
    return s;
}

#ifdef JAC_TILE2D_TYPE

template <typename R, int V, int RY>
static hipError_t t2_launch_s(const Geom &g, const void *uin, void *uout, const void *b,
                              double *res, double *gacc, const Tile2dPlan &pl, hipStream_t st) {
    T2Args A;
    A.t = pl.t;
    A.nstrips = pl.nstrips;
    A.ngrp = pl.ngrp;
    A.nitems = (int)pl.items;
    A.nt = pl.nt;
    A.acols = (pl.t + V - 1) / V * V;
#define JAC_T2(MODEV, RESV)                                                                     \
    hipLaunchKernelGGL((k_tile2d<R, V, RY, MODEV, RESV>), dim3((unsigned)pl.items),             \
                       dim3(64 * kT2Waves), 0, st, g, (const R *)uin, (R *)uout, (const R *)b,  \
                       res, gacc, A)
    if (gacc) {
        // the accumulator's registers: 16 cells per lane at most
        if constexpr (V * RY <= 16)
            JAC_T2(T2_ADJOINT, false);
        else
            return hipErrorInvalidValue;
    } else if (b && res)
        JAC_T2(T2_POISSON, true);
    else if (b)
        JAC_T2(T2_POISSON, false);
    else if (res)
        JAC_T2(T2_LAPLACE, true);
    else
        JAC_T2(T2_LAPLACE, false);
#undef JAC_T2
    return hipGetLastError();
}

template <typename R>
hipError_t t2_launch_r(const Geom &g, const void *uin, void *uout, const void *b, double *res,
                       double *gacc, const Tile2dPlan &pl, hipStream_t st) {
    switch (pl.shape) {
    case 0: return t2_launch_s<R, 1, 2>(g, uin, uout, b, res, gacc, pl, st);
    case 1: return t2_launch_s<R, 1, 4>(g, uin, uout, b, res, gacc, pl, st);
    case 2: return t2_launch_s<R, 2, 4>(g, uin, uout, b, res, gacc, pl, st);
    case 3: return t2_launch_s<R, 2, 8>(g, uin, uout, b, res, gacc, pl, st);
    case 4:
        if constexpr (sizeof(R) == 4)
            return t2_launch_s<R, 4, 8>(g, uin, uout, b, res, gacc, pl, st);
        return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}
template hipError_t t2_launch_r<JAC_TILE2D_TYPE>(const Geom &, const void *, void *, const void *,
                                                 double *, double *, const Tile2dPlan &,
                                                 hipStream_t);

#else  // dispatch object

// Tiles covering n cells when a tile of `hold` cells loses `halo` on each
// side that does not border the ring.
static int t2_tiles(int n, int hold, int halo) {
    const int out = hold - 2 * halo;
    return n <= hold ? 1 : out <= 0 ? 0 : (n - 2 * halo + out - 1) / out;
}

// Duration of a pass: kPassLaunchUs + its rounds of workgroups over the CUs x (c0 +
// c1 t, + cr with the residual) us, at least the time its bytes take, of which
// the part `mem` adds.  The figures per shape are fitted to passes of 1 .. 16
// sweeps timed on MI355X at 130^2 .. 8192^2 (FP32 sweeps: half of them within 6%);
// e.g. FP32 Poisson, 1000 x 777, 13 sweeps: 128 x 64 tiles 13.3 us,
// the marching pass 28.9; 2048^2: 256 x 128 tiles 32.4 us, marching 36.0; FP64
// 2500 x 1701, 13 sweeps: 128 x 128 tiles 51.4 us, marching (4 sweeps) 30.0;
// adjoint FP32 4096^2, 13 sweeps: 152 us, marching (7 sweeps) 105.7.  Shapes
// of at most 64 VGPRs run two workgroups per CU, which then take 3/4 of the
// time of two rounds; a last round counts in full among the first four
// (1000 x 777 adjoint, 1.2 workgroups per CU: 13 sweeps on 64 x 64 tiles 22.7 us, on
// 128 x 64 13.9).
struct T2Cost {
    double mem, c0, c1, cr;
    bool two;
};
static const T2Cost kT2Cost[2][3][5] = {
    // FP32: Laplace, Poisson, adjoint
    {{{1.64, 0.0, 0.19, 1.2, true}, {0.96, 0.0, 0.28, 1.1, true}, {0.21, 1.5, 0.30, 0.9, true}, {0, 2.1, 0.51, 4.1, false}, {0.25, 2.0, 1.14, 4.0, false}},
     {{1.42, 0.0, 0.19, 1.3, true}, {0.56, 0.3, 0.32, 1.4, true}, {0.21, 1.7, 0.34, 0.9, true}, {0.28, 3.0, 0.68, 2.8, false}, {0.42, 2.2, 1.40, 4.5, false}},
     {{0, 2.6, 0.22, 0, true}, {0, 3.3, 0.29, 0, true}, {0, 3.8, 0.55, 0, false}, {0, 5.9, 1.05, 0, false}, {0, 0, 0, 0, false}}},
    // FP64
    {{{0, 2.2, 0.27, 0, true}, {0, 2.8, 0.46, 0, true}, {0, 2.8, 0.62, 0, false}, {0, 4.8, 1.14, 0, false}, {0, 0, 0, 0, false}},
     {{0, 2.2, 0.27, 0, true}, {0, 2.8, 0.46, 0, true}, {0, 2.8, 0.62, 0, false}, {0, 4.8, 1.14, 0, false}, {0, 0, 0, 0, false}},
     {{0, 2.4, 0.30, 0, true}, {0, 3.2, 0.48, 0, true}, {0, 3.2, 0.70, 0, false}, {0, 5.7, 1.28, 0, false}, {0, 0, 0, 0, false}}},
};

template <typename R>
bool tile2d_plan(const Geom &g, int t, int mode, bool res, size_t cap, int cus, Tile2dPlan *out) {
    if (g.ndim != 2 || t < 1) return false;
    int ns;
    const T2Shape *sh = t2_shapes<R>(&ns);
    out->us = 1e300;
    const double cells = (double)g.n[0] * g.n[1];
    const double mem = cells * pass_bytes<R>(mode) / kPassBytesPerUs;
    for (int s = 0; s < ns; ++s) {
        if (mode == T2_ADJOINT && sh[s].v * sh[s].ry > 16) continue;
        Tile2dPlan p;
        p.t = t;
        p.shape = s;
        p.nt = 0;
        const int acols = (t + sh[s].v - 1) / sh[s].v * sh[s].v;
        p.nstrips = t2_tiles(g.n[0], 64 * sh[s].v, acols);
        p.ngrp = t2_tiles(g.n[1], kT2Waves * sh[s].ry, t);
        p.items = (int64_t)p.nstrips * p.ngrp;
        if (p.items <= 0 || p.items > 0x7fffffff || (res && (size_t)p.items > cap)) continue;
        const T2Cost &c = kT2Cost[sizeof(R) == 8][mode][s];
        const double full = (double)p.items / cus;
        const double whole = (double)((p.items + cus - 1) / cus);
        const double rounds = !c.two || full <= 1.0 ? whole : 0.75 * (full <= 4.0 ? whole : full);
        const double us = rounds * (c.c0 + c.c1 * t + (res ? c.cr : 0.0));
        const double add = c.mem * mem;
        p.us = kPassLaunchUs + add + (us > mem - add ? us : mem - add);
        if (p.us < out->us) *out = p;
    }
    return out->us < 1e300;
}

template <typename R>
hipError_t launch_tile2d(const Geom &g, const void *uin, void *uout, const void *b, double *res,
                         double *gacc, const Tile2dPlan &pl, hipStream_t st) {
    return t2_launch_r<R>(g, uin, uout, b, res, gacc, pl, st);
}

#define JAC_T2_DISPATCH(R)                                                                      \
    template bool tile2d_plan<R>(const Geom &, int, int, bool, size_t, int, Tile2dPlan *);      \
    template hipError_t launch_tile2d<R>(const Geom &, const void *, void *, const void *,      \
                                         double *, double *, const Tile2dPlan &, hipStream_t);
JAC_T2_DISPATCH(float)
JAC_T2_DISPATCH(double)

#endif  // JAC_TILE2D_TYPE

}  // namespace jac
