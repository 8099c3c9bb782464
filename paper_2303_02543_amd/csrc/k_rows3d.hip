// Pass kernel of 3D grids with one row per lane: up to four sweeps per pass, as
// k_march3d.hip, for the calls where it is the faster of the two (march3d_plan
// holds the rule).
//
// A workgroup of 8 waves holds 32 rows by 16 lanes of 16 bytes (one 16-lane row
// of a wave per grid row) and marches along z through a segment of planes.
// Each plane of the state and the source is loaded once, from whichever block
// owns it, and pushed through T levels: at the step that loads plane z + 1,
// level s computes plane z - s + 1 from the planes z - s .. z - s + 2 of level
// s - 1, three planes of every level in registers.  The rows y - 1 and y + 1
// of every level, the loaded planes' too, come from the LDS copy that level
// s - 1 wrote one step earlier (two buffers alternate by step, one barrier per
// step); x neighbours come from DPP shifts.  Level s is valid on the tile less
// s - 1 cells on every side.  Ring cells, and cells beyond the ring, copy
// their input at every level.
//
// What bounds it: memory (FP64 512^3 moves 3.2 GB per pass at depths 2 - 4 in the time
// of 2.8 TB/s, whatever the depth).  It is kept for what it measured against
// k_march3d.hip, whose loads per row are as many; the cause was not isolated.
// us per pass, it and the better of that kernel's tiles: FP64 512^3 Poisson, depth 2
// 1143 and 1214, depth 3 1147 and 1200, depth 4 1090 and 1162, but depth 5 1448 and
// 1108; 350x301x260 depths 2 - 3 254 - 262 and 231 - 234; 1024^2 x 3 depth 4 45 and 61;
// FP32 640^3 depth 1 Laplace 506 and 555, depth 2 764 and 884.  Deep-halo form,
// FP64 512^3 in 8^3 blocks, 60 sweeps at depth 4: 28.2 and 39.6 ms.
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "grid3d.h"
#include "jacobi_internal.h"
#include "kernels.h"

namespace jac {

constexpr int kR3Waves = 8;              // waves per work item (workgroup)
constexpr int kR3Threads = 64 * kR3Waves;
constexpr int kR3Rows = 4 * kR3Waves;    // rows held per work item (4 per wave)

template <typename R, int T>
struct R3 {
    static constexpr int V = 16 / (int)sizeof(R);
    static constexpr int W = 16 * V;                         // columns held per work item
    static constexpr int A0 = V * ((T - 1 + V - 1) / V);     // first output column (chunk-aligned)
    static constexpr int OW = V * ((W - (T - 1) - A0) / V);  // output columns per work item
    static constexpr int OY = kR3Rows - 2 * (T - 1);         // output rows per work item
    static constexpr int U = 6;   // steps per unrolled group: ring slots mod 3, LDS buffers mod 2
    static constexpr int NL = T > 1 ? T - 1 : 1;             // levels 1 .. T-1 held in registers
    static_assert(T >= 1 && T + 1 <= U, "source ring holds T + 1 planes");
    static_assert(OW > 0 && OY > 0, "tile too small for this depth");
};

// Plane cursor: global plane q (any integer), advanced one plane at a time;
// off / soff are the element offsets of plane q clamped to [-1, n_z] in the
// state buffers and (0 for the ring planes) in the source (the ring planes
// stand in for the planes beyond them).
struct R3Cur {
    int q, blk, loc;
    int64_t off, soff;
    __device__ __forceinline__ void set(const Geom &g) {
        off = plane_part(g, blk, loc);
        soff = q >= 0 && q < g.n[2] ? src_plane_part(g, blk, loc) : 0;
    }
    __device__ __forceinline__ void init(const Geom &g, int q0) {
        q = q0;
        owner(q0 < -1 ? -1 : q0 > g.n[2] ? g.n[2] : q0, g.e[2], g.nb[2], blk, loc);
        set(g);
    }
    __device__ __forceinline__ void advance(const Geom &g) {
        const bool moves = q >= -1 && q < g.n[2];
        ++q;
        if (moves) {
            ++loc;
            if (loc >= g.e[2] && blk < g.nb[2] - 1) {
                ++blk;
                loc = 0;
                set(g);
            } else {
                off += g.plane;
                soff = q >= 0 && q < g.n[2] ? (q == 0 ? src_plane_part(g, blk, loc)
                                                      : soff + (int64_t)g.e[1] * g.e[0])
                                            : 0;
            }
        }
    }
};

// Per-lane constants of a work item.
struct R3Lane {
    int64_t c_off, h_off, e_off, b_off;  // own row, halo row (loaders), edge cell, source
    int k;                               // LDS row slot of the lane's own row (1 .. 32)
    int hk;                              // LDS slot of the lane's halo load (0, 33; own slot: none)
    bool ld, lde, ldb;                   // lane loads interior/east-ring, edge, source
    bool upd[8];                         // element is an interior cell
    bool mine[8];                        // element is an output cell of this work item
    bool out_lane;                       // the whole chunk is output (interior tiles)
};

template <typename R, int T>
struct R3Regs {
    using S = R3<R, T>;
    Chunk<R, S::V> l0[3];       // level 0: planes by plane index mod 3
    Chunk<R, S::V> halo[3];     // level-0 halo row (loader lanes)
    R edge[3];                  // level-0 cell just outside the tile (row ends)
    Chunk<R, S::V> bq[S::U];    // source planes by plane index mod U
    Chunk<R, S::V> lv[S::NL][3];  // levels 1 .. T-1: planes by step mod 3
    double acc;                 // residual partial (level 1)
};

template <typename R, int T>
using R3Sh = Chunk<R, 16 / sizeof(R)> (*)[2][kR3Rows + 2][16];

// Store a register chunk into LDS element by element (one 16-byte write).
template <typename R, int V>
__device__ __forceinline__ void lds_put(Chunk<R, V> &dst, const Chunk<R, V> &src) {
    Chunk<R, V> t;
#pragma unroll
    for (int v = 0; v < V; ++v) t.v[v] = src.v[v];
    dst = t;
}

// Issue the loads of plane lc.q into slot J1 (level 0, halo, edge) and
// source slot JB, then advance the cursor.
template <typename R, int T, bool EDGE, bool SRC, int J1, int JB>
__device__ __forceinline__ void r3_load(const Geom &g, const R *__restrict__ uin,
                                        const R *__restrict__ bsrc, const R3Lane &L,
                                        R3Regs<R, T> &m, R3Cur &lc) {
    constexpr int V = R3<R, T>::V;
    using C = Chunk<R, V>;
    const int64_t pp = lc.off;
    // element-wise copies keep every ring slot in registers
    const C c = *reinterpret_cast<const C *>(uin + pp + L.c_off);
    // every lane loads (non-loader lanes their own row again), so no load
    // sits under a per-lane branch
    const C h = *reinterpret_cast<const C *>(uin + pp + L.h_off);
    const R e = uin[pp + L.e_off];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        m.l0[J1].v[v] = (EDGE && !L.ld) ? (R)0 : c.v[v];
        m.halo[J1].v[v] = (EDGE && !L.ld) ? (R)0 : h.v[v];
    }
    m.edge[J1] = (EDGE && !L.lde) ? (R)0 : e;
    if constexpr (SRC) {
        const C b = *reinterpret_cast<const C *>(bsrc + lc.soff + L.b_off);
#pragma unroll
        for (int v = 0; v < V; ++v) m.bq[JB].v[v] = (EDGE && !L.ldb) ? (R)0 : b.v[v];
    }
    lc.advance(g);
}

// Level S of step J (z = base + J): plane p = z - S + 1 of level S from the
// planes p-1, p, p+1 of level S-1 (registers) and the rows y-1, y+1 of plane
// p of level S-1 (LDS buffer J & 1).
template <typename R, int T, int MODE, bool EDGE, bool RES, int J, int S>
__device__ __forceinline__ void r3_level(const Geom &g, R *__restrict__ uout, const R3Lane &L,
                                         R3Regs<R, T> &m, R3Sh<R, T> sh, const int z,
                                         const int oz0, const int oz1, R3Cur &sc) {
    using M = R3<R, T>;
    constexpr int V = M::V;
    constexpr bool SRC = MODE == 1;
    using C = Chunk<R, V>;
    if constexpr (S <= T) {
        const int p = z - S + 1;
        const int cx = threadIdx.x & 15;
        C zm, zc, zp;
        R eo = (R)0;
        if constexpr (S == 1) {
            zm = m.l0[(J + 2) % 3];
            zc = m.l0[J % 3];
            zp = m.l0[(J + 1) % 3];
            eo = m.edge[J % 3];
        } else {
            zm = m.lv[S - 2][(J + 1) % 3];  // step J - 2
            zc = m.lv[S - 2][(J + 2) % 3];  // step J - 1
            zp = m.lv[S - 2][J % 3];        // this step
        }
        const C so = sh[S - 1][J & 1][L.k - 1][cx];
        const C no = sh[S - 1][J & 1][L.k + 1][cx];
        C bb;
        if constexpr (SRC) bb = m.bq[(J - S + 1 + M::U) % M::U];
        const R left = row_shift_up(eo, zc.v[V - 1]);
        const R right = row_shift_down(eo, zc.v[0]);
        const R w = (R)1 / (R)6;
        const bool pin = p >= 0 && p < g.n[2];
        const bool res_plane = RES && S == 1 && p >= oz0 && p < oz1;
        C out;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const R Wv = v > 0 ? zc.v[v - 1] : left;
            const R Ev = v < V - 1 ? zc.v[v + 1] : right;
            const R s = ((Wv + Ev) + (so.v[v] + no.v[v])) + (zm.v[v] + zp.v[v]);
            R o = SRC ? (s + bb.v[v]) * w : s * w;
            if (res_plane) {
                // residual of the input state, FP64 from widened values
                const double sd = (((double)Wv + (double)Ev) + ((double)so.v[v] + (double)no.v[v])) +
                                  ((double)zm.v[v] + (double)zp.v[v]);
                const double bd = SRC ? (double)bb.v[v] : 0.0;
                const double r = bd - (6.0 * (double)zc.v[v] - sd);
                m.acc += L.mine[v] ? r * r : 0.0;
            }
            // ring cells and cells beyond the ring keep their values
            if constexpr (EDGE) o = L.upd[v] ? o : zc.v[v];
            out.v[v] = o;
        }
        if (!pin) out = zc;  // a ring plane (or beyond) keeps its values
        if constexpr (S < T) {
            m.lv[S - 1][J % 3] = out;
        } else {
            if (uout && p >= oz0 && p < oz1) {
                R *q = uout + sc.off + L.c_off;
                if (!EDGE) {
                    if (L.out_lane) *reinterpret_cast<C *>(q) = out;
                } else {
#pragma unroll
                    for (int v = 0; v < V; ++v)
                        if (L.mine[v]) q[v] = out.v[v];
                }
            }
        }
        r3_level<R, T, MODE, EDGE, RES, J, S + 1>(g, uout, L, m, sh, z, oz0, oz1, sc);
    }
}

template <typename R, int T, int MODE, bool EDGE, bool RES, int J>
__device__ __forceinline__ void r3_steps(const Geom &g, const R *__restrict__ uin,
                                         R *__restrict__ uout, const R *__restrict__ bsrc,
                                         const R3Lane &L, R3Regs<R, T> &m, R3Sh<R, T> sh,
                                         const int base, const int zend, const int oz0,
                                         const int oz1, R3Cur &lc, R3Cur &sc) {
    using M = R3<R, T>;
    constexpr bool SRC = MODE == 1;
    if constexpr (J < M::U) {
        const int z = base + J;
        if (z > zend) return;
        const int cx = threadIdx.x & 15;
        // plane z + 1 of level 0, its halo row, edge cell and source
        r3_load<R, T, EDGE, SRC, (J + 1) % 3, (J + 1) % M::U>(g, uin, bsrc, L, m, lc);
        // level 0's plane z and levels 1 .. T-1's planes of the previous step
        // go to LDS buffer J & 1 for their y neighbours
        lds_put(sh[0][J & 1][L.k][cx], m.l0[J % 3]);
        lds_put(sh[0][J & 1][L.hk][cx], m.halo[J % 3]);  // non-loaders: their own row again
#pragma unroll
        for (int s = 1; s < T; ++s) lds_put(sh[s][J & 1][L.k][cx], m.lv[s - 1][(J + 2) % 3]);
        __syncthreads();
        r3_level<R, T, MODE, EDGE, RES, J, 1>(g, uout, L, m, sh, z, oz0, oz1, sc);
        sc.advance(g);
        r3_steps<R, T, MODE, EDGE, RES, J + 1>(g, uin, uout, bsrc, L, m, sh, base, zend, oz0, oz1,
                                               lc, sc);
    }
}

template <typename R, int T, int MODE, bool EDGE, bool RES>
__device__ __forceinline__ void r3_body(const Geom &g, const R *__restrict__ uin,
                                        R *__restrict__ uout, const R *__restrict__ bsrc,
                                        double *__restrict__ res_slot, const R3Lane &L, int oz0,
                                        int oz1, R3Sh<R, T> sh) {
    using M = R3<R, T>;
    constexpr int V = M::V;
    constexpr bool SRC = MODE == 1;
    R3Regs<R, T> m;
#pragma unroll
    for (int s = 0; s < M::NL; ++s)
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int v = 0; v < V; ++v) m.lv[s][k].v[v] = (R)0;
    m.acc = 0.0;
    // steps zs .. zend: level T computes planes oz0 .. oz1-1; planes zs-1 and
    // zs are loaded before the first step
    const int zs = oz0 - T + 1;
    const int zend = oz1 + T - 2;
    R3Cur lc, sc;
    lc.init(g, zs - 1);
    r3_load<R, T, EDGE, SRC, 2, M::U - 1>(g, uin, bsrc, L, m, lc);
    r3_load<R, T, EDGE, SRC, 0, 0>(g, uin, bsrc, L, m, lc);
    sc.init(g, zs - T + 1);  // the plane level T computes at the first step
    for (int base = zs; base <= zend; base += M::U)
        r3_steps<R, T, MODE, EDGE, RES, 0>(g, uin, uout, bsrc, L, m, sh, base, zend, oz0, oz1, lc,
                                           sc);
    if (RES) {
        const double a = wave_sum(m.acc);
        if ((threadIdx.x & 63) == 0) *res_slot = a;
    }
}

// Work item (one workgroup of 8 waves) number `item` of a grid cut into
// ngrp row groups (fastest), nstrips column strips and z segments of `zseg`
// output planes; wave q takes rows y0+4q .. y0+4q+3.  The residual partials
// are per wave: work item i owns partials 8i .. 8i+7 (res points at them).
template <typename R, int T, int MODE, bool RES>
__device__ __forceinline__ void r3_item(const Geom &g, const R *__restrict__ uin,
                                        R *__restrict__ uout, const R *__restrict__ bsrc,
                                        double *__restrict__ res, int item, int nstrips, int ngrp,
                                        int zseg, R3Sh<R, T> sh) {
    using M = R3<R, T>;
    constexpr int V = M::V;
    constexpr int W = M::W;
    const int grp = item % ngrp;
    const int rest = item / ngrp;
    const int strip = rest % nstrips;
    const int zs = rest / nstrips;
    const int wv = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int ry = lane >> 4, cx = lane & 15;
    const int nx = g.n[0], ny = g.n[1];
    const int a = strip * M::OW - M::A0;  // first column held
    const int c = a + cx * V;
    const int y0 = grp * M::OY - (T - 1);  // first row held
    const int kk = 4 * wv + ry;            // row within the tile
    const int yy = y0 + kk;
    auto clampy = [&](int y) { return y < -1 ? -1 : y > ny ? ny : y; };
    R3Lane L;
    L.k = 1 + kk;
    // chunk holds interior cells or ring / outside cells at in-bounds addresses
    L.ld = c <= nx;
    const int cl = L.ld ? c : 0;
    L.c_off = xy_part(g, cl, clampy(yy));
    L.hk = L.k;
    L.h_off = L.c_off;
    if (wv == 0 && ry == 0) {
        L.hk = 0;
        L.h_off = xy_part(g, cl, clampy(y0 - 1));
    } else if (wv == kR3Waves - 1 && ry == 3) {
        L.hk = kR3Rows + 1;
        L.h_off = xy_part(g, cl, clampy(y0 + kR3Rows));
    }
    // the first / last lane of each 16-lane row fetch the cells just west /
    // east of the tile; the others re-read their own first cell
    const int xe = cx == 0 ? a - 1 : cx == 15 ? a + W : c;
    L.lde = xe >= -1 && xe <= nx && (cx == 0 || cx == 15 || L.ld);
    L.e_off = xy_part(g, L.lde ? xe : 0, clampy(yy));
    const bool row_in = yy >= 0 && yy < ny;
    L.ldb = c >= 0 && c < nx && row_in;
    L.b_off = src_xy_part(g, L.ldb ? c : 0, L.ldb ? yy : 0);
    const bool out_row = kk >= T - 1 && kk < T - 1 + M::OY;
    L.out_lane = out_row && cx * V >= M::A0 && cx * V < M::A0 + M::OW;
#pragma unroll
    for (int v = 0; v < 8; ++v) {
        L.upd[v] = v < V && row_in && c + v >= 0 && c + v < nx;
        L.mine[v] = L.upd[v] && L.out_lane;
    }
    const int oz0 = zs * zseg;
    const int oz1 = oz0 + zseg < g.n[2] ? oz0 + zseg : g.n[2];
    double *slot = RES ? res + (int64_t)item * kR3Waves + wv : nullptr;
    const bool edge = a < 0 || a + W > nx || y0 < 0 || y0 + kR3Rows > ny;
    if (edge)
        r3_body<R, T, MODE, true, RES>(g, uin, uout, bsrc, slot, L, oz0, oz1, sh);
    else
        r3_body<R, T, MODE, false, RES>(g, uin, uout, bsrc, slot, L, oz0, oz1, sh);
}

// FP32 is compiled for four waves per SIMD, two workgroups per CU (left to
// itself the residual pass takes too many registers for the second).
template <typename R>
constexpr int r3_waves_per_simd() {
    return sizeof(R) == 4 ? 4 : 2;
}

template <typename R, int T, int MODE, bool RES>
__global__ __launch_bounds__(kR3Threads) __attribute__((amdgpu_waves_per_eu(r3_waves_per_simd<R>())))
void k_rows3d(Geom g, const R *__restrict__ uin,
                                                 R *__restrict__ uout,
                                                 const R *__restrict__ bsrc,
                                                 double *__restrict__ res, int nstrips, int ngrp,
                                                 int zseg, int nitems) {
    // per level 0 .. T-1: two plane buffers of rows y0-1 .. y0+kR3Rows
    __shared__ Chunk<R, R3<R, T>::V> sh[T][2][kR3Rows + 2][16];
    const int item = xcd_logical_block(blockIdx.x, gridDim.x);
    if (item >= nitems) return;  // whole workgroup
    r3_item<R, T, MODE, RES>(g, uin, uout, bsrc, res, item, nstrips, ngrp, zseg, sh);
}

// Batched pass: the work items of many grids in one launch (one descriptor
// each; the deep-halo form runs every block as its own grid).  Work item w
// belongs to grid gi with prefix[gi] <= w < prefix[gi+1]; every grid's input
// is u[0] and its output u[1].
template <typename R, int T, int MODE>
__global__ __launch_bounds__(kR3Threads) __attribute__((amdgpu_waves_per_eu(2)))
void k_rows3d_batch(const BatchGrid *__restrict__ grids,
                                                       const int *__restrict__ prefix,
                                                       int ngrids, int zseg, int nitems) {
    using M = R3<R, T>;
    __shared__ Chunk<R, M::V> sh[T][2][kR3Rows + 2][16];
    const int w = xcd_logical_block(blockIdx.x, gridDim.x);
    if (w >= nitems) return;  // whole workgroup
    int lo = 0, hi = ngrids;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (prefix[mid] <= w) lo = mid; else hi = mid;
    }
    const int gi = lo;
    const Geom g = grids[gi].g;
    const int nstrips = (g.n[0] + M::OW - 1) / M::OW;
    const int ngrp = (g.n[1] + M::OY - 1) / M::OY;
    r3_item<R, T, MODE, false>(g, (const R *)grids[gi].u[0], (R *)grids[gi].u[1],
                               (const R *)grids[gi].b, nullptr, w - prefix[gi], nstrips, ngrp, zseg,
                               sh);
}

template <typename R>
static void r3_shape(const Geom &g, int depth, int zseg, int &nstrips, int &ngrp, int &nzs) {
    auto of = [&](int ow, int oy) {
        nstrips = (g.n[0] + ow - 1) / ow;
        ngrp = (g.n[1] + oy - 1) / oy;
    };
    switch (depth) {
    case 1: of(R3<R, 1>::OW, R3<R, 1>::OY); break;
    case 2: of(R3<R, 2>::OW, R3<R, 2>::OY); break;
    case 3: of(R3<R, 3>::OW, R3<R, 3>::OY); break;
    case 4: of(R3<R, 4>::OW, R3<R, 4>::OY); break;
    default: of(R3<R, 5>::OW, R3<R, 5>::OY); break;
    }
    nzs = (g.n[2] + zseg - 1) / zseg;
}

template <typename R>
bool rows3d_plan(const Geom &g, int depth, int zseg, size_t cap, M3Plan *p) {
    if (depth < 1 || depth > kRows3dMaxDepth) return false;
    M3Plan r;
    r.row = true;
    r.wide = true;
    r.ry = 1;
    // output planes per work item unless set: shorter segments repeat the
    // 2 (T - 1) warm-up planes more often, longer ones leave too few work items
    r.zseg = zseg > 0 ? zseg : sizeof(R) == 4 ? 32 : 64;
    int nzs;
    r3_shape<R>(g, depth, r.zseg, r.nstrips, r.ngrp, nzs);
    r.items = (int64_t)r.nstrips * r.ngrp * nzs;
    r.partials = kR3Waves * r.items;
    if ((size_t)r.partials > cap || r.partials > 0x7fffffff - 3) return false;
    *p = r;
    return true;
}
template bool rows3d_plan<float>(const Geom &, int, int, size_t, M3Plan *);
template bool rows3d_plan<double>(const Geom &, int, int, size_t, M3Plan *);

int64_t rows3d_batch_items(const Geom &g, int zseg, int depth) {
    if (depth < 1 || depth > march3d_max_depth()) return -1;
    int ns, ng, nz;
    r3_shape<double>(g, depth, zseg, ns, ng, nz);
    return (int64_t)ns * ng * nz;
}

template <typename R, int T>
static hipError_t r3_launch(const Geom &g, const R *uin, R *uout, const R *b, double *res,
                            const M3Plan &pl, hipStream_t st) {
#define JAC_R3(MODEV, RESV)                                                                      \
    hipLaunchKernelGGL((k_rows3d<R, T, MODEV, RESV>), dim3((unsigned)pl.items), dim3(kR3Threads), \
                       0, st, g, uin, uout, b, res, pl.nstrips, pl.ngrp, pl.zseg, (int)pl.items)
    if (b && res)
        JAC_R3(1, true);
    else if (b)
        JAC_R3(1, false);
    else if (res)
        JAC_R3(0, true);
    else
        JAC_R3(0, false);
#undef JAC_R3
    return hipGetLastError();
}

template <typename R>
hipError_t launch_rows3d(const Geom &g, const void *uin, void *uout, const void *b, double *res,
                         const M3Plan &pl, hipStream_t st, int depth) {
    const R *u = (const R *)uin, *s = (const R *)b;
    R *o = (R *)uout;
    static_assert(kRows3dMaxDepth == 4, "depths below");
    switch (depth) {
    case 1: return r3_launch<R, 1>(g, u, o, s, res, pl, st);
    case 2: return r3_launch<R, 2>(g, u, o, s, res, pl, st);
    case 3: return r3_launch<R, 3>(g, u, o, s, res, pl, st);
    case 4: return r3_launch<R, 4>(g, u, o, s, res, pl, st);
    default: return hipErrorInvalidValue;
    }
}
template hipError_t launch_rows3d<float>(const Geom &, const void *, void *, const void *, double *,
                                         const M3Plan &, hipStream_t, int);
template hipError_t launch_rows3d<double>(const Geom &, const void *, void *, const void *, double *,
                                          const M3Plan &, hipStream_t, int);

template <int T>
static hipError_t r3b_launch(const BatchGrid *grids, const int *prefix, int ngrids, bool src,
                             int zseg, int nitems, hipStream_t st) {
    if (nitems <= 0) return hipSuccess;
    if (src)
        hipLaunchKernelGGL((k_rows3d_batch<double, T, 1>), dim3(nitems), dim3(kR3Threads), 0, st,
                           grids, prefix, ngrids, zseg, nitems);
    else
        hipLaunchKernelGGL((k_rows3d_batch<double, T, 0>), dim3(nitems), dim3(kR3Threads), 0, st,
                           grids, prefix, ngrids, zseg, nitems);
    return hipGetLastError();
}

hipError_t launch_rows3d_batch(const BatchGrid *grids, const int *prefix, int ngrids, bool src,
                               int depth, int zseg, int nitems, hipStream_t st) {
    switch (depth) {
    case 1: return r3b_launch<1>(grids, prefix, ngrids, src, zseg, nitems, st);
    case 2: return r3b_launch<2>(grids, prefix, ngrids, src, zseg, nitems, st);
    case 3: return r3b_launch<3>(grids, prefix, ngrids, src, zseg, nitems, st);
    case 4: return r3b_launch<4>(grids, prefix, ngrids, src, zseg, nitems, st);
    case 5: return r3b_launch<5>(grids, prefix, ngrids, src, zseg, nitems, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace jac
