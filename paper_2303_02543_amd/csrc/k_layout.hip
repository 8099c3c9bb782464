// Layout kernels: scatter a full state into blocks, gather it back, scale the
// source into blocks, and the face-halo exchange between blocks.
//
// The paper's proxy cuts the domain into cuboids and, every iteration, packs
// each block's edge cells, moves them to the face neighbours and unpacks them
// into their halos (Section 4.3; the over-decomposition timeline figure of
// Section 4.4 names the six per-face halo buffers).  On one GPU every block
// lives in the same HBM, so pack, copy and unpack collapse into one gather
// per halo cell: read the neighbour's edge cell, write the halo slot.
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "jacobi_internal.h"
#include "kernels.h"

namespace jac {

// The element maps below run over the rows of the blocks: a workgroup takes
// rows of one block plane (2D: of the block), `lanes` lanes per row, each lane
// V = 16 bytes of it, so that narrow blocks (64 columns of a 3D domain) fill
// the lanes as well as wide ones, and the block's side is read and written in
// aligned 16-byte pieces (the full array's rows have any alignment, which
// global 16-byte accesses take at 4 bytes).  Blocks, planes and rows come from
// the grid's coordinates, so no element needs a division.  Bound by memory;
// 512^3 FP32 in 64^3 blocks, before (one workgroup per row of the full array,
// a quarter of its lanes busy in each block) and now: scatter 664 us plus 464
// for the two halo exchanges it now includes -> 604; gather 548 -> 286; source
// 444 -> 203.  8192^2 FP32 in 512^2 blocks: 167 + 42 -> 154, 125 -> 88, 124 -> 100.
//
// Planes of fewer rows than a workgroup's lanes cover share one, as many planes as
// fit: 256^3 FP32 in 8^3-cell blocks, a plane per workgroup (16 of its 256 threads
// busy) and now: source 272 -> 48 us, gather 388 -> 155.
struct RowMap {
    int lanes, rows;  // lanes per row, rows per plane and step (both powers of two)
    dim3 grid;        // x: row groups, y: groups of planes, z: blocks (all strided beyond the limits)
};
// nrows, nplanes: rows per block plane and planes per block to cover
template <typename R>
static RowMap row_map(const Geom &g, int nrows, int nplanes) {
    constexpr int V = 16 / (int)sizeof(R);
    RowMap m;
    m.lanes = 1;
    while (m.lanes < 256 && m.lanes * V < g.e[0]) m.lanes *= 2;
    m.rows = 1;
    while (m.rows < 256 / m.lanes && m.rows < nrows) m.rows *= 2;
    const int per = 256 / (m.lanes * m.rows), pgroups = (nplanes + per - 1) / per;
    // up to four pieces per thread where that still leaves 1024 workgroups (2000x1500
    // FP64 gather, a workgroup per row 12.3 us, four rows each 9.5; a 256^2 gather
    // in one step each 3.5 us, in four 5.7), two in grids beyond the 256 MiB cache
    // (512^3 FP32 in 64^3 blocks, gather 324 us with four, 305 with two)
    int groups = (nrows + m.rows - 1) / m.rows;
    const double cells = (double)g.n[0] * g.n[1] * (g.ndim == 3 ? g.n[2] : 1);
    const int along = (g.e[0] + m.lanes * V - 1) / (m.lanes * V);
    const int most = (cells * sizeof(R) >= 268435456.0 ? 2 : 4) / along;
    const double fit = (double)groups * pgroups * (double)g.nblocks / 1024.0;
    const int steps = most < 1 || fit < 1.0 ? 1 : fit < most ? (int)fit : most;
    groups = (groups + steps - 1) / steps;
    m.grid = dim3((unsigned)(groups < 1 ? 1 : groups > (1 << 20) ? (1 << 20) : groups), (unsigned)(pgroups < 65535 ? pgroups : 65535),
                  (unsigned)(g.nblocks < 65535 ? g.nblocks : 65535));
    return m;
}

// A thread's lane, row and plane in its workgroup's step.
struct RowThread {
    int lane, row, plane;
    int nrows, nplanes;  // rows and planes that the grid covers in a step
    __device__ __forceinline__ RowThread(int lanes, int rows) {
        const int t = (int)threadIdx.x, per = 256 / (lanes * rows);
        lane = t & (lanes - 1);
        row = (int)blockIdx.x * rows + ((t / lanes) & (rows - 1));
        plane = (int)blockIdx.y * per + t / (lanes * rows);
        nrows = (int)gridDim.x * rows;
        nplanes = (int)gridDim.y * per;
    }
};

// 16 bytes at the full array's alignment
template <typename R>
struct __attribute__((packed, aligned(sizeof(R)))) Loose {
    R v[16 / sizeof(R)];
};

// A block's coordinates and extents.
struct BlockPos {
    int b[3], ext[3];
};
__device__ __forceinline__ BlockPos block_pos(const Geom &g, int64_t blk) {
    // fewer than 2^31 blocks (each stores at least 1 KiB): 32-bit divisions
    BlockPos p;
    const unsigned row = (unsigned)blk / (unsigned)g.nb[0];
    p.b[0] = (int)((unsigned)blk - row * g.nb[0]);
    p.b[2] = g.ndim == 3 ? (int)(row / (unsigned)g.nb[1]) : 0;
    p.b[1] = (int)row - p.b[2] * g.nb[1];
    for (int a = 0; a < 3; ++a) p.ext[a] = a < g.ndim ? extent(g.n[a], g.e[a], p.b[a]) : 1;
    return p;
}

// Every block's interior and one-cell frame from the full (n+2)^d array, in
// both state buffers: a frame cell holds the neighbour's value, or the
// Dirichlet ring on the domain's sides, so no halo exchange has to follow.
// zero_ring: the ring is written as 0.
template <typename R>
__global__ __launch_bounds__(256) void k_scatter(Geom g, const R *__restrict__ u,
                                                 R *__restrict__ s0, R *__restrict__ s1, int lanes,
                                                 int rows, int zero_ring) {
    constexpr int V = 16 / (int)sizeof(R);
    const int64_t nx2 = g.n[0] + 2, ny2 = g.n[1] + 2;
    const RowThread rt(lanes, rows);
    const int lz0 = g.ndim == 3 ? -1 : 0;
    for (int64_t blk = blockIdx.z; blk < g.nblocks; blk += gridDim.z) {
        const BlockPos p = block_pos(g, blk);
        const int ex = p.ext[0], ey = p.ext[1], hz = g.ndim == 3 ? p.ext[2] : 0;
        const int x0 = p.b[0] * g.e[0], y0 = p.b[1] * g.e[1], z0 = p.b[2] * g.e[2];
        for (int lz = lz0 + rt.plane; lz <= hz; lz += rt.nplanes) {
            const int z = z0 + lz;
            const bool zr = g.ndim == 3 && (z < 0 || z >= g.n[2]);
            for (int ly = -1 + rt.row; ly <= ey; ly += rt.nrows) {
                const int y = y0 + ly;
                const bool ring = zero_ring && (zr || y < 0 || y >= g.n[1]);
                const R *src = u + ((g.ndim == 3 ? (int64_t)(z + 1) * ny2 : 0) + y + 1) * nx2 + 1 + x0;
                const int64_t o = local_offset(g, blk, 0, ly, lz);
                for (int c = rt.lane * V; c < ex; c += lanes * V) {
                    if (c + V <= ex) {
                        Loose<R> t = *reinterpret_cast<const Loose<R> *>(src + c);
                        Chunk<R, V> w;
#pragma unroll
                        for (int v = 0; v < V; ++v) w.v[v] = ring ? (R)0 : t.v[v];
                        *reinterpret_cast<Chunk<R, V> *>(s0 + o + c) = w;
                        *reinterpret_cast<Chunk<R, V> *>(s1 + o + c) = w;
                    } else {
                        for (int v = 0; c + v < ex; ++v)
                            s0[o + c + v] = s1[o + c + v] = ring ? (R)0 : src[c + v];
                    }
                }
                // the cells west and east of the row
                if (rt.lane < 2) {
                    const int lx = rt.lane == 0 ? -1 : ex, x = x0 + lx;
                    const bool zero = ring || (zero_ring && (x < 0 || x >= g.n[0]));
                    s0[o + lx] = s1[o + lx] = zero ? (R)0 : src[lx];
                }
            }
        }
    }
}

// Every block's interior, and the ring nodes its frame holds on the domain's
// sides, to the full array.
template <typename R>
__global__ __launch_bounds__(256) void k_gather(Geom g, const R *__restrict__ s,
                                                R *__restrict__ u, int lanes, int rows) {
    constexpr int V = 16 / (int)sizeof(R);
    const int64_t nx2 = g.n[0] + 2, ny2 = g.n[1] + 2;
    const RowThread rt(lanes, rows);
    for (int64_t blk = blockIdx.z; blk < g.nblocks; blk += gridDim.z) {
        const BlockPos p = block_pos(g, blk);
        const int ex = p.ext[0];
        const int x0 = p.b[0] * g.e[0], y0 = p.b[1] * g.e[1], z0 = p.b[2] * g.e[2];
        // rows and planes of the frame on the domain's sides
        const int ylo = p.b[1] == 0 ? -1 : 0, yhi = p.ext[1] - (p.b[1] == g.nb[1] - 1 ? 0 : 1);
        int zlo = 0, zhi = 0;
        if (g.ndim == 3) {
            zlo = p.b[2] == 0 ? -1 : 0;
            zhi = p.ext[2] - (p.b[2] == g.nb[2] - 1 ? 0 : 1);
        }
        for (int lz = zlo + rt.plane; lz <= zhi; lz += rt.nplanes) {
            for (int ly = ylo + rt.row; ly <= yhi; ly += rt.nrows) {
                R *dst = u + ((g.ndim == 3 ? (int64_t)(z0 + lz + 1) * ny2 : 0) + y0 + ly + 1) * nx2 + 1 + x0;
                const int64_t o = local_offset(g, blk, 0, ly, lz);
                for (int c = rt.lane * V; c < ex; c += lanes * V) {
                    if (c + V <= ex) {
                        const Chunk<R, V> w = *reinterpret_cast<const Chunk<R, V> *>(s + o + c);
                        Loose<R> t;
#pragma unroll
                        for (int v = 0; v < V; ++v) t.v[v] = w.v[v];
                        *reinterpret_cast<Loose<R> *>(dst + c) = t;
                    } else {
                        for (int v = 0; c + v < ex; ++v) dst[c + v] = s[o + c + v];
                    }
                }
                if (rt.lane == 0 && p.b[0] == 0) dst[-1] = s[o - 1];
                if (rt.lane == 0 && p.b[0] == g.nb[0] - 1) dst[ex] = s[o + ex];
            }
        }
    }
}

// b = fl_R(h2 * f): the product in FP64, one rounding to R.
template <typename R>
__global__ __launch_bounds__(256) void k_scale_source(Geom g, const R *__restrict__ f,
                                                      R *__restrict__ b, double h2, int lanes,
                                                      int rows) {
    constexpr int V = 16 / (int)sizeof(R);
    const int64_t nx = g.n[0], ny = g.n[1];
    const RowThread rt(lanes, rows);
    for (int64_t blk = blockIdx.z; blk < g.nblocks; blk += gridDim.z) {
        const BlockPos p = block_pos(g, blk);
        const int ex = p.ext[0], ey = p.ext[1], ez = p.ext[2];
        const int x0 = p.b[0] * g.e[0], y0 = p.b[1] * g.e[1], z0 = p.b[2] * g.e[2];
        for (int lz = rt.plane; lz < ez; lz += rt.nplanes) {
            for (int ly = rt.row; ly < ey; ly += rt.nrows) {
                const R *src = f + ((int64_t)(z0 + lz) * ny + y0 + ly) * nx + x0;
                R *dst = b + blk * g.sstride + ((int64_t)lz * g.e[1] + ly) * g.e[0];
                for (int c = rt.lane * V; c < ex; c += lanes * V) {
                    if (c + V <= ex) {
                        const Loose<R> t = *reinterpret_cast<const Loose<R> *>(src + c);
                        Chunk<R, V> w;
#pragma unroll
                        for (int v = 0; v < V; ++v) w.v[v] = (R)(h2 * (double)t.v[v]);
                        *reinterpret_cast<Chunk<R, V> *>(dst + c) = w;
                    } else {
                        for (int v = 0; c + v < ex; ++v) dst[c + v] = (R)(h2 * (double)src[c + v]);
                    }
                }
            }
        }
    }
}

// Cell t of a face of a block along AXIS (the lower of the two tangential axes
// fastest, so y- and z-faces are contiguous rows): its place in the block at
// normal coordinate `at`, and in the block across the face at `nat`; false
// beyond the face.
template <int AXIS>
__device__ __forceinline__ bool face_cell(const Geom &g, const BlockPos &p, int64_t blk,
                                          int64_t nbr, int t, int at, int nat, int64_t *here,
                                          int64_t *there) {
    constexpr int TA = AXIS == 0 ? 1 : 0, TB = AXIS == 2 ? 1 : 2;
    const int fa = p.ext[TA];
    int hi = 0, lo = t;
    if (g.ndim == 3) {
        hi = t / fa;
        lo = t - hi * fa;
        if (hi >= p.ext[TB]) return false;
    } else if (t >= fa) {
        return false;
    }
    int l[3] = {0, 0, 0}, m[3] = {0, 0, 0};
    l[TA] = m[TA] = lo;
    l[TB] = m[TB] = hi;
    l[AXIS] = at;
    m[AXIS] = nat;
    *here = local_offset(g, blk, l[0], l[1], l[2]);
    *there = local_offset(g, nbr, m[0], m[1], m[2]);
    return true;
}

// Cell t of the faces of block blk along AXIS.  SEND: the block's edge cell goes
// into the halo of its face neighbour; otherwise the block's halo takes the
// neighbour's edge cell.  SIDES = 2: of both faces (low, high), else of face
// `side0`.
template <typename R, int AXIS, bool SEND, int SIDES>
__device__ __forceinline__ void face_copy(const Geom &g, R *__restrict__ s, int64_t blk,
                                          const BlockPos &p, int side0, int t) {
    const int64_t step = AXIS == 0 ? 1 : AXIS == 1 ? g.nb[0] : (int64_t)g.nb[0] * g.nb[1];
    int64_t to[SIDES];
    bool in[SIDES];
    R v[SIDES];
#pragma unroll
    for (int q = 0; q < SIDES; ++q) {
        const int side = SIDES == 2 ? q : side0;
        const bool ring = side == 0 ? p.b[AXIS] == 0 : p.b[AXIS] == g.nb[AXIS] - 1;
        const int64_t nbr = side == 0 ? blk - step : blk + step;
        // a low neighbour is a full block
        const int at = SEND ? (side == 0 ? 0 : p.ext[AXIS] - 1) : (side == 0 ? -1 : p.ext[AXIS]);
        const int nat = SEND ? (side == 0 ? g.e[AXIS] : -1) : (side == 0 ? g.e[AXIS] - 1 : 0);
        int64_t here = 0, there = 0;
        // a face on the domain's side keeps the Dirichlet ring
        in[q] = !ring && face_cell<AXIS>(g, p, blk, nbr, t, at, nat, &here, &there);
        to[q] = SEND ? there : here;
        if (in[q]) v[q] = s[SEND ? here : there];
    }
#pragma unroll
    for (int q = 0; q < SIDES; ++q)
        if (in[q]) s[to[q]] = v[q];
}

// Halo exchange (SEND = false) of every block, or the face sends of the
// blocks b0 .. b1-1: sending the faces of every block fills the same halo
// cells, with the same values, as the exchange.  Faces on the domain boundary
// keep the Dirichlet values.
//
// The west and east halo cells of a row lie in one 128-byte line (the end of
// one stored row and the start of the next), so a workgroup fills both x-faces of
// a block: from two, mostly on different XCDs, every line was written twice.
//
// PACK: faces of at most 128 cells, `lanes` threads each, consecutive groups of
// threads on consecutive faces of a block (exchange alone, a workgroup per face
// and now: 4096^2 FP32 in 32^2 blocks 46.4 -> 31.2 us, 16^2 94 -> 53, 64^2 24.6 -> 16.7;
// one thread after the other over all faces, with a division each: 32.3, 54, 18.2).
// Otherwise a thread does one cell of a face, or of both faces of an axis
// (SIDES), and the grid runs over a face's cells, the axes and the blocks.  In 2D
// the axes come last: faces of one axis may fill few of the workgroups that the
// longest face needs, and workgroups of one axis, dealt out in between, then
// sit on the same XCDs (2048^2 FP32 in 32 x 1024 blocks 11.0 us, axes last 6.6).
// In 3D the axes of a block come one after the other (512^3 in 64^3 blocks 236 us,
// axes last 256).  The faces of a 3D block are sent one by one: they go to
// different blocks, and an overlapped sweep of 256^3 FP32 in 32^3 blocks takes 131 us,
// 134 with both from one thread; 2D sends of 8 columns by 4096 rows 765 and 812
// the other way round.
template <typename R, bool SEND, bool PACK, int SIDES>
__global__ __launch_bounds__(256) void k_halo(Geom g, R *__restrict__ s, int64_t b0, int64_t b1,
                                              int lanes, int64_t stride) {
    if constexpr (PACK) {
        const int sub = (int)threadIdx.x / lanes, per = 256 / lanes, t0 = (int)threadIdx.x % lanes;
        // launched with at most 2^30 groups of threads
        const unsigned nf = g.ndim == 3 ? 6 : 4;
        const unsigned i0 = blockIdx.x * per + sub;
        const unsigned rel0 = g.ndim == 3 ? i0 / 6u : i0 / 4u, face = i0 - rel0 * nf;
        const unsigned axis = face >> 1, side = face & 1;
        for (int64_t blk = b0 + rel0; blk < b1; blk += stride) {
            const BlockPos p = block_pos(g, blk);
            if (axis == 0)
                face_copy<R, 0, SEND, SIDES>(g, s, blk, p, side, t0);
            else if (axis == 1)
                face_copy<R, 1, SEND, SIDES>(g, s, blk, p, side, t0);
            else
                face_copy<R, 2, SEND, SIDES>(g, s, blk, p, side, t0);
        }
    } else {
        const int t0 = (int)(blockIdx.x * 256 + threadIdx.x);
        const int face = (int)(g.ndim == 3 ? blockIdx.y : blockIdx.z) * SIDES;
        const int axis = face >> 1, side = face & 1;
        for (int64_t blk = b0 + (int64_t)(g.ndim == 3 ? blockIdx.z : blockIdx.y); blk < b1;
             blk += stride) {
            const BlockPos p = block_pos(g, blk);
            if (axis == 0)
                face_copy<R, 0, SEND, SIDES>(g, s, blk, p, side, t0);
            else if (axis == 1)
                face_copy<R, 1, SEND, SIDES>(g, s, blk, p, side, t0);
            else
                face_copy<R, 2, SEND, SIDES>(g, s, blk, p, side, t0);
        }
    }
}

static inline int grid_for(int64_t total) {
    int64_t b = (total + 255) / 256;
    if (b > 65536) b = 65536;
    if (b < 1) b = 1;
    return (int)b;
}

template <typename R>
hipError_t launch_scatter(const Geom &g, const void *u, void *s0, void *s1, bool zero_ring,
                          hipStream_t st) {
    const RowMap m = row_map<R>(g, g.e[1] + 2, g.ndim == 3 ? g.e[2] + 2 : 1);
    hipLaunchKernelGGL(k_scatter<R>, m.grid, dim3(256), 0, st, g, (const R *)u, (R *)s0, (R *)s1,
                       m.lanes, m.rows, zero_ring ? 1 : 0);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_fill_f64(double *__restrict__ p, double v, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

hipError_t launch_fill_f64(double *p, double v, int64_t n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_f64, dim3(grid_for(n)), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}

// End of a 2D adjoint run.  gb: FP64 interior accumulator dL/db (n_y x n_x).
// Two stream-ordered kernels so that grad_f may alias gb:
//  1. grad_ring (full (n_y+2) x (n_x+2) array): each non-corner ring node gets
//     gb at the one interior node next to it (dL/dg_q = sum_k w lam_k[p(q)]
//     = gb[p(q)]); corners and interior nodes get 0;
//  2. grad_f (interior) = h2 * gb.
__global__ __launch_bounds__(256) void k_adjoint_ring(int nx, int ny, const double *__restrict__ gb,
                                                      double *__restrict__ grad_ring,
                                                      int64_t total) {
    const int64_t nx2 = nx + 2;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int x = (int)(i % nx2) - 1;
        const int y = (int)(i / nx2) - 1;
        const bool inx = x >= 0 && x < nx, iny = y >= 0 && y < ny;
        double v = 0.0;
        if (inx && !iny) v = gb[(int64_t)(y < 0 ? 0 : ny - 1) * nx + x];
        if (iny && !inx) v = gb[(int64_t)y * nx + (x < 0 ? 0 : nx - 1)];
        grad_ring[i] = v;
    }
}

// Full dL/dU0 of a 2D adjoint run whose loss reads all of u_K (ring
// included).  A sweep copies the ring, so the ring of u_K is g itself and
// each ring node gets dL/du_K there plus, for non-corner nodes, what flowed
// through the sweeps (gb at its interior neighbour); corners get only
// dL/du_K.  Interior nodes get lam_0, read from the blocked state s.
template <typename R>
__global__ __launch_bounds__(256) void k_adjoint_full(Geom g, const double *__restrict__ gb,
                                                      const R *__restrict__ lamK,
                                                      const R *__restrict__ s,
                                                      double *__restrict__ out, int64_t total) {
    const int nx = g.n[0], ny = g.n[1];
    const int64_t nx2 = nx + 2;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int x = (int)(i % nx2) - 1;
        const int y = (int)(i / nx2) - 1;
        const bool inx = x >= 0 && x < nx, iny = y >= 0 && y < ny;
        double v;
        if (inx && iny) {
            v = (double)s[state_offset(g, x, y, 0)];
        } else {
            v = (double)lamK[i];
            if (inx) v = v + gb[(int64_t)(y < 0 ? 0 : ny - 1) * nx + x];
            if (iny) v = v + gb[(int64_t)y * nx + (x < 0 ? 0 : nx - 1)];
        }
        out[i] = v;
    }
}

template <typename R>
hipError_t launch_adjoint_full(const Geom &g, const double *gb, const void *lamK, const void *s,
                               double *out, hipStream_t st) {
    const int64_t total = (int64_t)(g.n[0] + 2) * (g.n[1] + 2);
    hipLaunchKernelGGL(k_adjoint_full<R>, dim3(grid_for(total)), dim3(256), 0, st, g, gb,
                       (const R *)lamK, (const R *)s, out, total);
    return hipGetLastError();
}
template hipError_t launch_adjoint_full<float>(const Geom &, const double *, const void *,
                                               const void *, double *, hipStream_t);
template hipError_t launch_adjoint_full<double>(const Geom &, const double *, const void *,
                                                const void *, double *, hipStream_t);

__global__ __launch_bounds__(256) void k_scale_f64(const double *gb, double h2, double *out,
                                                   int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = h2 * gb[i];
}

hipError_t launch_adjoint_finish(const Geom &g, const double *gb, double h2, double *grad_f,
                                 double *grad_ring, hipStream_t st) {
    if (grad_ring) {
        const int64_t total = (int64_t)(g.n[0] + 2) * (g.n[1] + 2);
        hipLaunchKernelGGL(k_adjoint_ring, dim3(grid_for(total)), dim3(256), 0, st, g.n[0],
                           g.n[1], gb, grad_ring, total);
    }
    if (grad_f) {
        const int64_t n = (int64_t)g.n[0] * g.n[1];
        hipLaunchKernelGGL(k_scale_f64, dim3(grid_for(n)), dim3(256), 0, st, gb, h2, grad_f, n);
    }
    return hipGetLastError();
}

template <typename R>
hipError_t launch_gather(const Geom &g, const void *s, void *u, hipStream_t st) {
    const RowMap m = row_map<R>(g, g.e[1] + 2, g.ndim == 3 ? g.e[2] + 2 : 1);
    hipLaunchKernelGGL(k_gather<R>, m.grid, dim3(256), 0, st, g, (const R *)s, (R *)u, m.lanes,
                       m.rows);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_scale_source(const Geom &g, const void *f, void *b, double h2, hipStream_t st) {
    const RowMap m = row_map<R>(g, g.e[1], g.ndim == 3 ? g.e[2] : 1);
    hipLaunchKernelGGL(k_scale_source<R>, m.grid, dim3(256), 0, st, g, (const R *)f, (R *)b, h2,
                       m.lanes, m.rows);
    return hipGetLastError();
}

// The faces of blocks b0 .. b1-1.
template <typename R, bool SEND>
static hipError_t launch_faces(const Geom &g, void *s, int64_t b0, int64_t b1, hipStream_t st) {
    // the longest face between blocks (an axis of one block has none)
    int64_t m = 0;
    for (int a = 0; a < g.ndim; ++a) {
        const int64_t face = (int64_t)g.e[a == 0 ? 1 : 0] * g.e[a == 2 ? 1 : 2];
        if (g.nb[a] > 1 && face > m) m = face;
    }
    if (m == 0) return hipSuccess;
    if (m > 0x7fffffff - 4096) return hipErrorInvalidValue;
    const int64_t blocks = b1 - b0;
    if (m <= 128) {
        int lanes = 4;
        while (lanes < m) lanes *= 2;
        // whole blocks per step of the grid, so that a thread's face is fixed
        const int nf = 2 * g.ndim, per = 256 / lanes;
        const int64_t most = (1 << 28) / nf;
        const int64_t stride = blocks < most ? blocks : most;
        hipLaunchKernelGGL((k_halo<R, SEND, true, 1>), dim3((unsigned)((stride * nf + per - 1) / per)),
                           dim3(256), 0, st, g, (R *)s, b0, b1, lanes, stride);
        return hipGetLastError();
    }
    const unsigned cells = (unsigned)((m + 255) / 256);
    const unsigned strided = (unsigned)(blocks < 65535 ? blocks : 65535);
    if (g.ndim == 2)
        hipLaunchKernelGGL((k_halo<R, SEND, false, 2>), dim3(cells, strided, 2), dim3(256), 0, st, g,
                           (R *)s, b0, b1, 256, (int64_t)strided);
    else if constexpr (SEND)
        hipLaunchKernelGGL((k_halo<R, true, false, 1>), dim3(cells, 6, strided), dim3(256), 0, st, g,
                           (R *)s, b0, b1, 256, (int64_t)strided);
    else
        hipLaunchKernelGGL((k_halo<R, false, false, 2>), dim3(cells, 3, strided), dim3(256), 0, st, g,
                           (R *)s, b0, b1, 256, (int64_t)strided);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_halo_exchange(const Geom &g, void *s, hipStream_t st) {
    if (g.nblocks <= 1) return hipSuccess;  // no internal face
    return launch_faces<R, false>(g, s, 0, g.nblocks, st);
}

template <typename R>
hipError_t launch_halo_send(const Geom &g, void *s, int64_t b0, int64_t b1, hipStream_t st) {
    if (b1 <= b0) return hipSuccess;
    return launch_faces<R, true>(g, s, b0, b1, st);
}

template hipError_t launch_halo_send<float>(const Geom &, void *, int64_t, int64_t, hipStream_t);
template hipError_t launch_halo_send<double>(const Geom &, void *, int64_t, int64_t, hipStream_t);
template hipError_t launch_scatter<float>(const Geom &, const void *, void *, void *, bool,
                                          hipStream_t);
template hipError_t launch_scatter<double>(const Geom &, const void *, void *, void *, bool,
                                           hipStream_t);
template hipError_t launch_gather<float>(const Geom &, const void *, void *, hipStream_t);
template hipError_t launch_gather<double>(const Geom &, const void *, void *, hipStream_t);
template hipError_t launch_scale_source<float>(const Geom &, const void *, void *, double, hipStream_t);
template hipError_t launch_scale_source<double>(const Geom &, const void *, void *, double, hipStream_t);
template hipError_t launch_halo_exchange<float>(const Geom &, void *, hipStream_t);
template hipError_t launch_halo_exchange<double>(const Geom &, void *, hipStream_t);

}  // namespace jac
