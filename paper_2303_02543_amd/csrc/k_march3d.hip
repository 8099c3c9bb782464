// Fused 3D Jacobi pass kernel for gfx950: T sweeps per pass (temporal
// blocking along z), halo cells read straight from the neighbouring blocks,
// and the FP64 residual of the pass's input state folded into the first
// level.
//
// The update is the 7-point Jacobi step of the proxy application in
// Section 4.3 of the paper, evaluated as
//   s = ((W + E) + (S + N)) + (B + F);  u' = (s + b) * fl(1/6)
// with no FMA contraction, so every schedule gives the same bits.
//
// A workgroup of 8 waves holds a tile of 64 (FP32) / 32 (FP64) columns by
// H = 32 RY rows and marches along z through a segment of planes.  A lane holds
// 16 bytes of RY consecutive rows; 16 lanes span the tile's width and a wave 4 RY rows.  Each
// plane of the state and the source is loaded from whichever block owns it
// -- the exchange of halo cells between blocks happens inside these loads --
// and pushed through T levels: at step z, level s computes plane z - s + 1
// from the planes z - s .. z - s + 2 of level s - 1, held in registers.
// x neighbours come from DPP shifts within each 16-lane row, y neighbours
// from the lane's own rows and, at its first and last row, from the LDS copy
// of level s - 1's boundary rows that their lanes wrote one step earlier (two
// buffers alternate by step, one barrier per step serves every level).
// Level 1 reads the rows just outside a lane's own from memory instead (the
// L1 holds them: the neighbouring lane loads the same rows), so its
// arithmetic runs before the barrier.  Level s is valid on the tile less
// s - 1 cells on every side, except where the tile ends at the domain's ring:
// there the ring values (x: the lane's edge cell; y: the halo rows of the
// LDS buffers, handed from level to level) keep every level valid up to the
// ring.  So the first and last tile of an axis need no halo beyond the ring,
// and k tiles of 64 columns at depth 5 cover 56 k + 8 columns.
//
// A segment that ends in the middle of an unrolled group ends the wave there:
// leaving through the loop would merge the register rings of the group's
// steps (copies of every plane, and waits for the loads in flight).
//
// What bounds it: memory.  The state's plane z + 2, and the source, edge cells
// and outer rows of plane z + 1, are requested at step z and used one step
// later, and a step takes 2.6 us whatever the depth (512^3 FP32, one workgroup
// per CU: depth 3 467 us per pass, depth 4 464, depth 5 470, 4.1 TB/s of counter
// traffic, 1.25x the algorithmic bytes).  So the deepest pass and the largest
// tile the registers and the LDS hold win: 64 rows at two rows per lane, one
// workgroup of 8 waves per CU.  Smaller tiles with two workgroups per CU (32
// rows: 724 us at depth 5), loads two steps ahead (475 us) and non-temporal
// stores (516 us) were slower.  Per pass of 512^3 (this kernel at depth 5, and
// the kernel of 32-row tiles without prefetch at depth 4 before it): FP32 1428
// and 856 G updates/s, FP64 608 and 480.
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "grid3d.h"
#include "jacobi_internal.h"
#include "kernels.h"

namespace jac {

constexpr int kM3Waves = 8;              // waves per work item (workgroup)
constexpr int kM3Threads = 64 * kM3Waves;

template <typename R, int T, int RY>
struct M3 {
    static constexpr int V = 16 / (int)sizeof(R);            // columns per lane
    static constexpr int W = 16 * V;                         // columns held per work item
    static constexpr int H = 4 * RY * kM3Waves;              // rows held per work item
    static constexpr int A0 = V * ((T - 1 + V - 1) / V);     // halo columns (chunk-aligned)
    static constexpr int OW = W - 2 * A0;                    // output columns of an inner strip
    static constexpr int OY = H - 2 * (T - 1);               // output rows of an inner row group
    static constexpr int U = 6;   // steps per unrolled group: plane slots mod 6 / 3 / 2
    static constexpr int NL = T > 1 ? T - 1 : 1;             // levels 1 .. T-1 held in registers
    static_assert(T >= 1 && T + 1 <= U, "source ring holds T + 1 planes");
    static_assert(OW > 0 && OY > 0, "tile too small for this depth");
};

// LDS copies of levels 1 .. T-1: [level][step parity][row + 1][lane of the row]
template <typename R, int T, int RY>
using M3Sh = Chunk<R, M3<R, T, RY>::V> (*)[2][M3<R, T, RY>::H + 2][16];

// Plane cursor: global plane q (any integer), advanced one plane at a time;
// off / soff are the element offsets of plane q clamped to [-1, n_z] in the
// state buffers and to [0, n_z - 1] in the source.  Moving into the next
// block layer adds the layer's step less the planes already counted.
struct ZCur {
    int q, loc, left;  // global plane, plane within the block, blocks after this one
    int64_t off, soff;
    __device__ __forceinline__ void init(const Geom &g, int q0) {
        q = q0;
        int blk;
        owner(q0 < -1 ? -1 : q0 > g.n[2] ? g.n[2] : q0, g.e[2], g.nb[2], blk, loc);
        left = g.nb[2] - 1 - blk;
        off = plane_part(g, blk, loc);
        int sblk, sloc;
        owner(q0 < 0 ? 0 : q0 > g.n[2] - 1 ? g.n[2] - 1 : q0, g.e[2], g.nb[2], sblk, sloc);
        soff = src_plane_part(g, sblk, sloc);
    }
    __device__ __forceinline__ void advance(const Geom &g) {
        const int64_t layer = (int64_t)g.nb[1] * g.nb[0];
        const int64_t splane = (int64_t)g.e[1] * g.e[0];
        const bool moves = q >= -1 && q < g.n[2];
        const bool smoves = q >= 0 && q < g.n[2] - 1;
        const bool wrap = loc + 1 >= g.e[2] && left > 0;
        const int64_t d = wrap ? layer * g.bstride - (g.e[2] - 1) * g.plane : g.plane;
        const int64_t sd = wrap ? layer * g.sstride - (g.e[2] - 1) * splane : splane;
        off += moves ? d : 0;
        soff += smoves ? sd : 0;
        loc = moves ? (wrap ? 0 : loc + 1) : loc;
        left -= moves && wrap ? 1 : 0;
        ++q;
    }
};

// Per-lane constants of a work item.  Offsets are bytes from the start of a
// plane; OFF is 32 bits unless a z layer of blocks spans 4 GiB or more.
template <typename OFF, int RY>
struct M3Lane {
    OFF c[RY], up, dn, e[RY], b[RY];  // own rows, rows y-1 / y+1, edge cells, source rows
    uint32_t st[RY];                  // own rows' whole-chunk stores (kNoStore: none)
    int lr, cx;                       // LDS row slot of the first own row, lane within the row
    int nxr;                          // interior columns from the lane's first on (EDGE)
    int nyr;                          // interior rows from the lane's first on (EDGE)
    int o0, o1;                       // own rows [o0, o1) are outputs (0 .. RY)
    bool out_lane;                    // the lane's columns are outputs (EDGE: those < nxr)
    bool ylo, yhi;                    // lane keeps the ring row below / above its rows
    bool wring;                       // the wave has such lanes (uniform)
};

template <typename R, int T, int RY>
struct M3Regs {
    using S = M3<R, T, RY>;
    R l0[S::U][RY][S::V];      // level 0: planes by plane mod 6 (four live)
    R up[2][S::V], dn[2][S::V];  // level 0: rows y-1 / y+1 by plane mod 2
    R ed[S::U][RY];            // level 0: cell just outside the tile (row ends)
    R bq[S::U][RY][S::V];      // source planes by plane mod 6
    R lv[S::NL][2][RY][S::V];  // levels 1 .. T-1: the two newest planes, by step mod 2
    R zm[2][RY][S::V];         // the plane before them, read back from LDS, by level mod 2
    R so[2][S::V], no[2][S::V];  // outer rows read from LDS, by level mod 2
    int64_t off[S::U];         // state offsets of planes z - T + 1 .. z + 2, by plane mod 6
    double acc;                // residual partial (level 1)
};

// A lane's chunk / cell at byte offset `off` from a uniform base.  32-bit
// offsets go through a buffer descriptor of the plane (scalar base, vector
// offset): no address arithmetic and one register per offset.
template <typename R, int V, typename OFF>
__device__ __forceinline__ void m3_get(R (&dst)[V], const R *base, OFF off) {
    Chunk<R, V> t;
    if constexpr (sizeof(OFF) == 4)
        t = buffer_get<Chunk<R, V>>(base, off);
    else
        t = *reinterpret_cast<const Chunk<R, V> *>(reinterpret_cast<const char *>(base) + off);
#pragma unroll
    for (int v = 0; v < V; ++v) dst[v] = t.v[v];
}
template <typename R, typename OFF>
__device__ __forceinline__ R m3_get1(const R *base, OFF off) {
    if constexpr (sizeof(OFF) == 4)
        return buffer_get<R>(base, off);
    else
        return *reinterpret_cast<const R *>(reinterpret_cast<const char *>(base) + off);
}

// Own rows of the cursor's plane into plane slot S6, then advance.
template <typename R, int T, int RY, int S6, typename OFF>
__device__ __forceinline__ void m3_load_own(const Geom &g, const R *__restrict__ uin,
                                            const M3Lane<OFF, RY> &L, M3Regs<R, T, RY> &m,
                                            ZCur &lc) {
    m.off[S6] = lc.off;
    const R *p = uin + lc.off;
#pragma unroll
    for (int j = 0; j < RY; ++j) m3_get<R, M3<R, T, RY>::V>(m.l0[S6][j], p, L.c[j]);
    lc.advance(g);
}

// Outer rows, edge cells and source of the plane at (off, soff) into slots.
template <typename R, int T, int RY, bool SRC, int S6, int S2, typename OFF>
__device__ __forceinline__ void m3_load_rest(const R *__restrict__ uin,
                                             const R *__restrict__ bsrc, int64_t off,
                                             int64_t soff, const M3Lane<OFF, RY> &L,
                                             M3Regs<R, T, RY> &m) {
    const R *p = uin + off;
    m3_get<R, M3<R, T, RY>::V>(m.up[S2], p, L.up);
    m3_get<R, M3<R, T, RY>::V>(m.dn[S2], p, L.dn);
#pragma unroll
    for (int j = 0; j < RY; ++j)
        m.ed[S6][j] = m3_get1<R>(p, L.e[j]);
    if constexpr (SRC) {
#pragma unroll
        for (int j = 0; j < RY; ++j) m3_get<R, M3<R, T, RY>::V>(m.bq[S6][j], bsrc + soff, L.b[j]);
    }
}

template <typename R, int V>
__device__ __forceinline__ void lds_put(Chunk<R, V> &dst, const R (&src)[V]) {
    Chunk<R, V> t;
#pragma unroll
    for (int v = 0; v < V; ++v) t.v[v] = src[v];
    dst = t;
}
template <typename R, int V>
__device__ __forceinline__ void lds_get(const Chunk<R, V> &src, R (&dst)[V]) {
    const Chunk<R, V> t = src;
#pragma unroll
    for (int v = 0; v < V; ++v) dst[v] = t.v[v];
}

// What level S takes from LDS: the outer rows of plane z - S + 1 of level
// S - 1, written one step ago, and the lane's own rows of plane z - S, written
// two steps ago (kept there instead of in registers: a level then holds two
// planes, not three).  Read one
// level ahead of their use, so that the LDS latency overlaps the arithmetic of
// the level in between, and before level S - 1 overwrites plane z - S.
template <typename R, int T, int RY, int J, int S, typename OFF>
__device__ __forceinline__ void m3_read_rows(const M3Lane<OFF, RY> &L, M3Regs<R, T, RY> &m,
                                             M3Sh<R, T, RY> sh) {
    constexpr int V = M3<R, T, RY>::V;
    lds_get<R, V>(sh[S - 2][J & 1][L.lr - 1][L.cx], m.so[S & 1]);
    lds_get<R, V>(sh[S - 2][J & 1][L.lr + RY][L.cx], m.no[S & 1]);
#pragma unroll
    for (int j = 0; j < RY; ++j)
        lds_get<R, V>(sh[S - 2][(J + 1) & 1][L.lr + j][L.cx], m.zm[S & 1][j]);
}

// Level S of step J (z = base + J): plane p = z - S + 1 of level S from the
// planes p-1, p, p+1 of level S-1.  EDGE: the tile holds ring columns or rows,
// or its first / last column borders the ring.
template <typename R, int T, int RY, int MODE, bool EDGE, bool RES, int J, int S,
          typename OFF>
__device__ __forceinline__ void m3_level(const Geom &g, R *__restrict__ uout,
                                         const M3Lane<OFF, RY> &L, M3Regs<R, T, RY> &m,
                                         M3Sh<R, T, RY> sh, const int z, const int oz0,
                                         const int oz1, const int64_t out_off) {
    using M = M3<R, T, RY>;
    constexpr int V = M::V, U = M::U;
    constexpr bool SRC = MODE == 1;
    if constexpr (S <= T) {
        const int p = z - S + 1;
        constexpr int SP = (J - S + 1 + U) % U;  // slot of plane p (level 0 data)
        R zm[RY][V], zc[RY][V], zp[RY][V], so[V], no[V];
#pragma unroll
        for (int j = 0; j < RY; ++j)
#pragma unroll
            for (int v = 0; v < V; ++v) {
                if constexpr (S == 1) {
                    zm[j][v] = m.l0[(J + U - 1) % U][j][v];
                    zc[j][v] = m.l0[J % U][j][v];
                    zp[j][v] = m.l0[(J + 1) % U][j][v];
                } else {
                    zm[j][v] = m.zm[S & 1][j][v];               // step J - 2
                    zc[j][v] = m.lv[S - 2][(J + 1) % 2][j][v];  // step J - 1
                    zp[j][v] = m.lv[S - 2][J % 2][j][v];        // this step
                }
            }
        if constexpr (S == 1) {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                so[v] = m.up[J % 2][v];
                no[v] = m.dn[J % 2][v];
            }
        } else {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                so[v] = m.so[S & 1][v];
                no[v] = m.no[S & 1][v];
            }
            if constexpr (S < T) {
                m3_read_rows<R, T, RY, J, S + 1>(L, m, sh);
                // keep the reads ahead of this level's arithmetic
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        const R w = (R)1 / (R)6;
        const bool res_plane = RES && S == 1 && p >= oz0 && p < oz1;
        R out[RY][V];
#pragma unroll
        for (int j = 0; j < RY; ++j) {
            // the cell outside the tile: needed by level 1, and by every
            // level where it is the domain's ring
            const R eo = (S == 1 || EDGE) ? m.ed[SP][j] : (R)0;
            const R left = row_shift_up(eo, zc[j][V - 1]);
            const R right = row_shift_down(eo, zc[j][0]);
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const R Wv = v > 0 ? zc[j][v - 1] : left;
                const R Ev = v < V - 1 ? zc[j][v + 1] : right;
                const R Sv = j > 0 ? zc[j - 1][v] : so[v];
                const R Nv = j < RY - 1 ? zc[j + 1][v] : no[v];
                const R s = ((Wv + Ev) + (Sv + Nv)) + (zm[j][v] + zp[j][v]);
                R o = SRC ? (s + m.bq[SP][j][v]) * w : s * w;
                if constexpr (RES && S == 1) {
                    if (res_plane) {
                        // residual of the input state, FP64 from widened values
                        const double sd = (((double)Wv + (double)Ev) + ((double)Sv + (double)Nv)) +
                                          ((double)zm[j][v] + (double)zp[j][v]);
                        const double bd = SRC ? (double)m.bq[SP][j][v] : 0.0;
                        const double r = bd - (6.0 * (double)zc[j][v] - sd);
                        const bool mine = L.out_lane && j >= L.o0 && j < L.o1 &&
                                          (!EDGE || v < L.nxr);
                        m.acc += mine ? r * r : 0.0;
                    }
                }
                // ring cells and cells beyond the ring keep their values
                if constexpr (EDGE) o = (v < L.nxr && j < L.nyr) ? o : zc[j][v];
                out[j][v] = o;
            }
        }
        // the empty asm keeps the arithmetic above in one block with its DPP
        // shifts; without it the compiler moves it under the test below and
        // cannot fold the shifts into the additions
#pragma unroll
        for (int j = 0; j < RY; ++j)
#pragma unroll
            for (int v = 0; v < V; ++v) asm("" : "+v"(out[j][v]));
        if (__builtin_expect(p < 0 || p >= g.n[2], 0)) {  // a ring plane (or beyond) keeps its values
#pragma unroll
            for (int j = 0; j < RY; ++j)
#pragma unroll
                for (int v = 0; v < V; ++v) out[j][v] = zc[j][v];
        }
        if constexpr (S < T) {
#pragma unroll
            for (int j = 0; j < RY; ++j)
#pragma unroll
                for (int v = 0; v < V; ++v) m.lv[S - 1][J % 2][j][v] = out[j][v];
        } else {
            const bool on = uout && p >= oz0 && p < oz1;
            if constexpr (sizeof(OFF) == 4) {
#pragma unroll
                for (int j = 0; j < RY; ++j) {
                    Chunk<R, V> t;
#pragma unroll
                    for (int v = 0; v < V; ++v) t.v[v] = out[j][v];
                    buffer_put16(uout + out_off, L.st[j], on, t);
                }
            }
            // chunks that hold the east ring column are stored cell by cell
            // (with 64-bit offsets, every chunk)
            if (on && L.out_lane && (sizeof(OFF) != 4 || (EDGE && L.nxr < V))) {
                R *q = uout + out_off;
#pragma unroll
                for (int j = 0; j < RY; ++j) {
                    if (j < L.o0 || j >= L.o1) continue;
                    R *d = reinterpret_cast<R *>(reinterpret_cast<char *>(q) + L.c[j]);
#pragma unroll
                    for (int v = 0; v < V; ++v)
                        if (v < L.nxr) d[v] = out[j][v];
                }
            }
        }
        if constexpr (S == 1 && T > 1) {
            __syncthreads();
            m3_read_rows<R, T, RY, J, 2>(L, m, sh);
        }
        if constexpr (S < T) {
            // this plane's boundary rows for the neighbouring lanes' next
            // step; where the tile ends at the ring in y, also the ring row,
            // handed on from this level's own neighbour row
            auto &rows = sh[S - 1][(J + 1) & 1];
            if constexpr (RY > 1) lds_put<R, V>(rows[L.lr + RY - 1][L.cx], out[RY - 1]);
            lds_put<R, V>(rows[L.lr][L.cx], out[0]);
            if (L.wring) {
                if (L.ylo) lds_put<R, V>(rows[L.lr - 1][L.cx], so);
                if (L.yhi) lds_put<R, V>(rows[L.lr + RY][L.cx], no);
            }
        }
        m3_level<R, T, RY, MODE, EDGE, RES, J, S + 1>(g, uout, L, m, sh, z, oz0, oz1, out_off);
    }
}

template <typename R, int T, int RY, int MODE, bool EDGE, bool RES, int J,
          typename OFF>
__device__ __forceinline__ void m3_steps(const Geom &g, const R *__restrict__ uin,
                                         R *__restrict__ uout, const R *__restrict__ bsrc,
                                         double *__restrict__ res_slot,
                                         const M3Lane<OFF, RY> &L, M3Regs<R, T, RY> &m,
                                         M3Sh<R, T, RY> sh, const int base, const int zend,
                                         const int oz0, const int oz1, ZCur &lc, int64_t &soff1) {
    using M = M3<R, T, RY>;
    constexpr bool SRC = MODE == 1;
    constexpr int U = M::U;
    if constexpr (J < U) {
        const int z = base + J;
        if (z > zend) {
            if constexpr (RES) {
                const double a = wave_sum(m.acc);
                if ((threadIdx.x & 63) == 0) *res_slot = a;
            }
            __builtin_amdgcn_endpgm();
        }
        // the cursor is at plane z + 2; soff1 is plane z + 1
        const int64_t out_off = m.off[(J - T + 1 + U) % U], soff2 = lc.soff;
        m3_load_rest<R, T, RY, SRC, (J + 1) % U, (J + 1) % 2>(uin, bsrc, m.off[(J + 1) % U], soff1,
                                                             L, m);
        m3_load_own<R, T, RY, (J + 2) % U>(g, uin, L, m, lc);
        soff1 = soff2;
        m3_level<R, T, RY, MODE, EDGE, RES, J, 1>(g, uout, L, m, sh, z, oz0, oz1, out_off);
        m3_steps<R, T, RY, MODE, EDGE, RES, J + 1>(g, uin, uout, bsrc, res_slot, L, m, sh, base,
                                                  zend, oz0, oz1, lc, soff1);
    }
}

template <typename R, int T, int RY, int MODE, bool EDGE, bool RES, typename OFF>
__device__ __forceinline__ void m3_body(const Geom &g, const R *__restrict__ uin,
                                        R *__restrict__ uout, const R *__restrict__ bsrc,
                                        double *__restrict__ res_slot, const M3Lane<OFF, RY> &L,
                                        int oz0, int oz1, M3Sh<R, T, RY> sh) {
    using M = M3<R, T, RY>;
    constexpr int V = M::V, U = M::U;
    constexpr bool SRC = MODE == 1;
    M3Regs<R, T, RY> m;
#pragma unroll
    for (int s = 0; s < M::NL; ++s)
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int j = 0; j < RY; ++j)
#pragma unroll
                for (int v = 0; v < V; ++v) m.lv[s][k][j][v] = (R)0;
    m.acc = 0.0;
#pragma unroll
    for (int k = 0; k < U; ++k)
#pragma unroll
        for (int j = 0; j < RY; ++j) {
            m.ed[k][j] = (R)0;
#pragma unroll
            for (int v = 0; v < V; ++v) m.bq[k][j][v] = (R)0;
        }
    // steps zs .. zend: level T computes planes oz0 .. oz1-1; planes zs-1 ..
    // zs+1 and the rest of plane zs are loaded before the first step
    const int zs = oz0 - T + 1;
    const int zend = oz1 + T - 2;
    ZCur lc;
    lc.init(g, zs - 1);
#pragma unroll
    for (int k = 0; k < U; ++k) m.off[k] = lc.off;
    m3_load_own<R, T, RY, U - 1>(g, uin, L, m, lc);
    int64_t soff1 = lc.soff;
    m3_load_own<R, T, RY, 0>(g, uin, L, m, lc);
    m3_load_rest<R, T, RY, SRC, 0, 0>(uin, bsrc, m.off[0], soff1, L, m);
    soff1 = lc.soff;
    m3_load_own<R, T, RY, 1>(g, uin, L, m, lc);
    for (int base = zs;; base += U)
        m3_steps<R, T, RY, MODE, EDGE, RES, 0>(g, uin, uout, bsrc, res_slot, L, m, sh, base, zend,
                                              oz0, oz1, lc, soff1);
}

// Strips of columns and groups of rows covering n cells: `hold` cells held
// per tile, `out` of them outputs of an inner tile; the first and last tile
// also output the (hold - out) / 2 cells next to the ring.
__host__ __device__ inline int m3_tiles(int n, int hold, int out) {
    const int rest = n - (hold - out);
    return rest <= out ? 1 : (rest + out - 1) / out;
}

// Work item (one workgroup of 8 waves) number `item` of a grid cut into
// ngrp row groups (fastest), nstrips column strips and z segments of `zseg`
// output planes.  The residual partials are per wave: work item i owns
// partials 8i .. 8i+7 (res points at them).
template <typename R, int T, int RY, int MODE, bool RES, typename OFF>
__device__ __forceinline__ void m3_item(const Geom &g, const R *__restrict__ uin,
                                        R *__restrict__ uout, const R *__restrict__ bsrc,
                                        double *__restrict__ res, int item, int nstrips, int ngrp,
                                        int zseg, M3Sh<R, T, RY> sh) {
    using M = M3<R, T, RY>;
    constexpr int V = M::V, W = M::W, H = M::H;
    const int grp = item % ngrp;
    const int rest = item / ngrp;
    const int strip = rest % nstrips;
    const int zs = rest / nstrips;
    const int wv = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int ry = lane >> 4, cx = lane & 15;
    const int nx = g.n[0], ny = g.n[1];
    const int a = strip * M::OW;           // first column held
    const int c = a + cx * V;
    const int y0 = grp * M::OY;            // first row held
    const int kk = (4 * wv + ry) * RY;     // the lane's first row within the tile
    const int yy = y0 + kk;
    auto clampy = [&](int y) { return y < -1 ? -1 : y > ny ? ny : y; };
    M3Lane<OFF, RY> L;
    L.cx = cx;
    L.lr = 1 + kk;
    // chunk holds interior cells or ring / outside cells at in-bounds addresses
    const int cl = c <= nx ? c : 0;
    // the first / last lane of each 16-lane row fetch the cells just west /
    // east of the tile; the others re-read their own first cell
    const int xe = cx == 0 ? a - 1 : cx == 15 ? a + W : c;
    const int xel = xe <= nx ? xe : 0;
#pragma unroll
    for (int j = 0; j < RY; ++j) {
        const int y = clampy(yy + j);
        L.c[j] = (OFF)(xy_part(g, cl, y) * (int64_t)sizeof(R));
        L.e[j] = (OFF)(xy_part(g, xel, y) * (int64_t)sizeof(R));
        const bool lb = c < nx && yy + j < ny;
        L.b[j] = (OFF)(src_xy_part(g, lb ? c : 0, lb ? yy + j : 0) * (int64_t)sizeof(R));
    }
    L.up = (OFF)(xy_part(g, cl, clampy(yy - 1)) * (int64_t)sizeof(R));
    L.dn = (OFF)(xy_part(g, cl, clampy(yy + RY)) * (int64_t)sizeof(R));
    L.nxr = nx - c;
    L.nyr = ny - yy;
    // output rows and columns: less T-1 rows / A0 columns where the tile
    // continues beyond, up to the ring where it does not
    const int ylo = grp == 0 ? 0 : T - 1;
    const int yhi = grp == ngrp - 1 ? ny - y0 : H - (T - 1);
    L.o0 = ylo - kk;
    L.o1 = yhi - kk;
    const int xlo = strip == 0 ? 0 : M::A0;
    const int xhi = strip == nstrips - 1 ? nx - a : W - M::A0;
    L.out_lane = cx * V >= xlo && cx * V < xhi;
#pragma unroll
    for (int j = 0; j < RY; ++j)
        L.st[j] = L.out_lane && j >= L.o0 && j < L.o1 && L.nxr >= V ? (uint32_t)L.c[j] : kNoStore;
    // the ring row y = -1 lies just below the first tile, y = ny just above
    // a tile that ends with row ny - 1
    L.ylo = y0 == 0 && kk == 0;
    L.yhi = y0 + H == ny && kk + RY == H;
    L.wring = (y0 == 0 && wv == 0) || (y0 + H == ny && wv == kM3Waves - 1);
    const int oz0 = zs * zseg;
    const int oz1 = oz0 + zseg < g.n[2] ? oz0 + zseg : g.n[2];
    double *slot = RES ? res + (int64_t)item * kM3Waves + wv : nullptr;
    const bool edge = a == 0 || a + W >= nx || y0 + H > ny;
    if (edge)
        m3_body<R, T, RY, MODE, true, RES>(g, uin, uout, bsrc, slot, L, oz0, oz1, sh);
    else
        m3_body<R, T, RY, MODE, false, RES>(g, uin, uout, bsrc, slot, L, oz0, oz1, sh);
}

template <typename R, int T, int RY, int MODE, bool RES, typename OFF>
__global__ __launch_bounds__(kM3Threads) __attribute__((amdgpu_waves_per_eu(2)))
void k_march3d(Geom g, const R *__restrict__ uin, R *__restrict__ uout,
               const R *__restrict__ bsrc, double *__restrict__ res, int nstrips, int ngrp,
               int zseg, int nitems) {
    using M = M3<R, T, RY>;
    __shared__ Chunk<R, M::V> sh[M::NL][2][M::H + 2][16];
    const int item = xcd_logical_block(blockIdx.x, gridDim.x);
    if (item >= nitems) return;  // whole workgroup
    m3_item<R, T, RY, MODE, RES, OFF>(g, uin, uout, bsrc, res, item, nstrips, ngrp, zseg, sh);
}

// Batched pass: the work items of many grids in one launch (one descriptor
// each; the deep-halo form runs every block as its own grid).  Work item w
// belongs to grid gi with prefix[gi] <= w < prefix[gi+1]; every grid's input
// is u[0] and its output u[1].  FP32 on 32-row tiles, two workgroups per CU:
// 512^3 in 8^3 blocks of frames of 4, 60 sweeps at depth 5, 18.5 ms against 26.0
// on 64-row tiles (blocks of 72 rows: two tiles of 64 or three of 32) and 29.4
// for the row kernel of k_rows3d.hip, which runs FP64.
template <typename R, int T, int MODE, typename OFF>
__global__ __launch_bounds__(kM3Threads) __attribute__((amdgpu_waves_per_eu(2)))
void k_march3d_batch(const BatchGrid *__restrict__ grids, const int *__restrict__ prefix,
                     int ngrids, int zseg, int nitems) {
    using M = M3<R, T, 1>;
    __shared__ Chunk<R, M::V> sh[M::NL][2][M::H + 2][16];
    const int w = xcd_logical_block(blockIdx.x, gridDim.x);
    if (w >= nitems) return;  // whole workgroup
    int lo = 0, hi = ngrids;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (prefix[mid] <= w) lo = mid; else hi = mid;
    }
    const int gi = lo;
    const Geom g = grids[gi].g;
    const int nstrips = m3_tiles(g.n[0], M::W, M::OW);
    const int ngrp = m3_tiles(g.n[1], M::H, M::OY);
    m3_item<R, T, 1, MODE, false, OFF>(g, (const R *)grids[gi].u[0], (R *)grids[gi].u[1],
                                        (const R *)grids[gi].b, nullptr, w - prefix[gi], nstrips,
                                        ngrp, zseg, sh);
}

// ---- host side -------------------------------------------------------------
// The kernels of each depth T are compiled in an object of their own (this
// file built with JAC_MARCH3D_DEPTH=T); the object built without it holds the
// depth dispatch and the schedule rule.

template <typename R, int T>
hipError_t m3_launch_t(const Geom &g, const void *uin, void *uout, const void *b, double *res,
                       const M3Plan &pl, hipStream_t st);
template <int T>
hipError_t m3b_launch_t(const BatchGrid *grids, const int *prefix, int ngrids, bool src, bool wide,
                        int zseg, int nitems, hipStream_t st);

// Rows held per lane in the taller of the two tile heights (64 rows).
constexpr int kM3Ry = 2;

#ifdef JAC_MARCH3D_DEPTH

template <typename R, int T, int RY, typename OFF>
static hipError_t m3_launch_ry(const Geom &g, const void *uin, void *uout, const void *b,
                               double *res, const M3Plan &pl, hipStream_t st) {
    const int items = (int)pl.items;
    const R *bb = (const R *)b;
#define JAC_M3(MODEV, RESV)                                                                   \
    hipLaunchKernelGGL((k_march3d<R, T, RY, MODEV, RESV, OFF>), dim3(items), dim3(kM3Threads), 0, \
                       st, g, (const R *)uin, (R *)uout, bb, res, pl.nstrips, pl.ngrp, pl.zseg, \
                       items)
    if (b && res)
        JAC_M3(1, true);
    else if (b)
        JAC_M3(1, false);
    else if (res)
        JAC_M3(0, true);
    else
        JAC_M3(0, false);
#undef JAC_M3
    return hipGetLastError();
}

template <typename R, int T>
hipError_t m3_launch_t(const Geom &g, const void *uin, void *uout, const void *b, double *res,
                       const M3Plan &pl, hipStream_t st) {
    if (pl.wide) return m3_launch_ry<R, T, 1, uint64_t>(g, uin, uout, b, res, pl, st);
    if (pl.ry == kM3Ry)
        return m3_launch_ry<R, T, kM3Ry, uint32_t>(g, uin, uout, b, res, pl, st);
    return m3_launch_ry<R, T, 1, uint32_t>(g, uin, uout, b, res, pl, st);
}

template <int T>
hipError_t m3b_launch_t(const BatchGrid *grids, const int *prefix, int ngrids, bool src, bool wide,
                        int zseg, int nitems, hipStream_t st) {
    if (nitems <= 0) return hipSuccess;
#define JAC_M3B(MODEV, OFFV)                                                                     \
    hipLaunchKernelGGL((k_march3d_batch<float, T, MODEV, OFFV>), dim3(nitems), dim3(kM3Threads), \
                       0, st, grids, prefix, ngrids, zseg, nitems)
    if (wide && src)
        JAC_M3B(1, uint64_t);
    else if (wide)
        JAC_M3B(0, uint64_t);
    else if (src)
        JAC_M3B(1, uint32_t);
    else
        JAC_M3B(0, uint32_t);
#undef JAC_M3B
    return hipGetLastError();
}

#define JAC_M3_INSTANTIATE(R, T)                                                                \
    template hipError_t m3_launch_t<R, T>(const Geom &, const void *, void *, const void *,      \
                                          double *, const M3Plan &, hipStream_t);
JAC_M3_INSTANTIATE(float, JAC_MARCH3D_DEPTH)
JAC_M3_INSTANTIATE(double, JAC_MARCH3D_DEPTH)
template hipError_t m3b_launch_t<JAC_MARCH3D_DEPTH>(const BatchGrid *, const int *, int, bool, bool,
                                                    int, int, hipStream_t);

#else  // dispatch object

int march3d_max_depth() { return 5; }

// Tile counts of one pass at depth T with RY rows per lane.
template <typename R>
static void m3_shape(const Geom &g, int T, int ry, int &nstrips, int &ngrp) {
    const int v = 16 / (int)sizeof(R), w = 16 * v, h = 32 * ry;
    const int a0 = v * ((T - 1 + v - 1) / v);
    nstrips = m3_tiles(g.n[0], w, w - 2 * a0);
    ngrp = m3_tiles(g.n[1], h, h - 2 * (T - 1));
}

// The lane offsets of a plane are 32-bit byte offsets from the start of a
// z layer of blocks.
static bool m3_wide(const Geom &g, size_t es) {
    const double blk = (double)(g.bstride > g.sstride ? g.bstride : g.sstride);
    const double span = ((double)g.nb[0] * g.nb[1] - 1.0) * blk +
                        (double)(g.plane > (int64_t)g.e[0] * g.e[1] ? g.plane : (int64_t)g.e[0] * g.e[1]);
    return (span + g.ax + 64.0) * (double)es >= (double)kBufferBytes;
}

// Which tiles, and the row kernel or the tiles: by estimated time, per depth.
// The tiles' unit is a plane step of a 32-row tile per round of workgroups over
// the CUs; a step of a 64-row tile takes `tall` units, and plans of several
// rounds, which share less of their neighbours' planes in the L2s, `several`
// times as many.  A plane step of the row kernel per round, two workgroups per CU,
// takes `row` units (0: not compiled), its rounds counted whole below
// `whole_below` cells.  It is a choice from `least` cells on, on plates of up to 32
// planes from `plate` cells on, and is taken from `always` on.
//
// The constants are those that pick best among passes timed at 35 grids of 64^3 ..
// 640^3, plates, and bars, with and without source, and checked at 30 others: passes
// that are further than 5% behind the row kernel by itself are FP64 1024^2 x 3 at depth 1
// (14.4 and 12.8 us), and FP64 depth 5 of 1024^2 x 128 (1487 and 1386).  FP64 residuals alone, tiles and rows:
// 300x280x320 Laplace 68 and 54 us, 280^3 47 and 50.  us per pass, tiles and row
// kernel: FP64 512^3 Poisson depth 2 1200 and 1116, depth 4 1153 and 1071, but 640^3
// depth 2 1928 and 2307 (one round); 400^3 depth 2 532 and 501, 350x301x260 229 and 256;
// 1024^2 x 3 depth 4 61 and 45.  FP32 640^3 Laplace depth 1 555 and 506, depth 2 884 and
// 764, 600x520x500 depth 1 477 and 438, but 512^3 depth 2 454 and 554, 353x343x186 45 and 70.
struct M3Rule {
    double tall, several, row, whole_below, least, plate, always;
    double residual;  // `least` of passes without stores
};
constexpr double kNever = 1e300;
static const M3Rule kM3Rule[2][5] = {
    // FP32, depths 1 - 5
    {{1.9, 1.0, 1.85, kNever, 1.05e8, 1 << 21, 1.05e8, 6.2e7},
     {1.8, 1.2, 1.75, kNever, 1 << 26, kNever, kNever, kNever},
     {1.8, 1.1, 1.70, 0, 1 << 26, kNever, kNever, kNever},
     {1.8, 1.0, 1.60, kNever, 1 << 26, kNever, kNever, kNever},
     {1.8, 1.0, 0, 0, kNever, kNever, kNever, kNever}},
    // FP64
    {{1.8, 1.0, 1.75, 0, 5.5e7, kNever, kNever, 2.6e7},
     {1.8, 1.0, 1.40, kNever, 4e7, 0, kNever, kNever},
     {1.8, 1.2, 1.60, kNever, 4e7, 0, kNever, kNever},
     {1.8, 1.0, 1.48, 5e7, 0, 0, kNever, kNever},
     {1.8, 1.0, 0, 0, kNever, kNever, kNever, kNever}},
};

template <typename R>
bool march3d_plan(const Geom &g, int depth, int zseg, int cus, size_t cap, bool store, M3Plan *out) {
    if (depth < 1 || depth > march3d_max_depth()) return false;
    const M3Rule &rule = kM3Rule[sizeof(R) == 8][depth - 1];
    const int nz = g.n[2];
    M3Plan best;
    double best_cost = 1e300;
    const bool wide = m3_wide(g, sizeof(R));
    for (int ry = 1; ry <= (wide ? 1 : kM3Ry); ++ry) {
        M3Plan p;
        p.ry = ry;
        p.wide = wide;
        m3_shape<R>(g, depth, ry, p.nstrips, p.ngrp);
        const int64_t tiles = (int64_t)p.nstrips * p.ngrp;
        // (without stores 1.8: 256^3 FP32 Laplace residual, 32 rows 25.0 us, 64 rows 23.0)
        const double step = ry == 1 ? 1.0 : store ? rule.tall : 1.8;
        const int smin = zseg > 0 ? (nz + zseg - 1) / zseg : 1;
        const int smax = zseg > 0 ? smin : (nz + 3) / 4;
        for (int s = smin; s <= smax; ++s) {
            p.zseg = zseg > 0 ? zseg : (nz + s - 1) / s;
            const int64_t segs = (nz + p.zseg - 1) / p.zseg;
            p.items = tiles * segs;
            p.partials = kM3Waves * p.items;
            if ((size_t)p.partials > cap || p.partials > 0x7fffffff - 3) break;
            const int64_t rounds = (p.items + cus - 1) / cus;
            const double cost = rounds * step * (rounds > 1 ? rule.several : 1.0) *
                                (p.zseg + 2 * (depth - 1) + 3);
            if (cost < best_cost) {
                best_cost = cost;
                best = p;
            }
            if (rounds > 16) break;
        }
    }
    M3Plan row;
    if (rule.row > 0 && rows3d_plan<R>(g, depth, zseg, cap, &row)) {
        const double cells = (double)g.n[0] * g.n[1] * nz;
        const double full = (double)row.items / (2 * cus);
        const double rounds = cells < rule.whole_below ? (double)((row.items + 2 * cus - 1) / (2 * cus))
                                                       : full > 1.0 ? full : 1.0;
        const int planes = row.zseg < nz ? row.zseg : nz;
        const bool choice =
            cells >= (store ? rule.least : rule.residual) || (nz <= 32 && cells >= rule.plate);
        row.cost = rule.row * rounds * (planes + 2 * (depth - 1));
        // A sweep whose row tiles cover the grid with nothing over and fill a round of
        // one or of two workgroups per CU (residuals alone: of two) has no better
        // tiling; us, tiles and rows: FP32 512x256x256 Laplace 89 and 74, 256^3 29.1 and 26.4,
        // FP64 512x256x256 167 and 147; but with 320 of 512 workgroups, 320x256x256 FP64 119 and
        // 141, and with 4% over, 253x250x255 FP32 Laplace 32 and 52.
        const double fill = (double)row.items / cus;
        const bool whole = depth == 1 &&
                           (double)row.items * (256.0 / sizeof(R)) * 32 * row.zseg <= 1.02 * cells &&
                           ((store && fill > 0.875 && fill <= 1.0) ||
                            (fill > (store ? 1.74 : 1.95) && fill <= 2.0));
        if (whole || (choice && row.cost < best_cost) || cells >= rule.always || best_cost >= 1e300) {
            *out = row;
            return true;
        }
    }
    best.cost = best_cost;
    *out = best;
    return best_cost < 1e300;
}

#define JAC_M3_SWITCH(depth, F, ...)                  \
    switch (depth) {                                  \
    case 1: return JAC_M3_CASE(F, 1)(__VA_ARGS__);    \
    case 2: return JAC_M3_CASE(F, 2)(__VA_ARGS__);    \
    case 3: return JAC_M3_CASE(F, 3)(__VA_ARGS__);    \
    case 4: return JAC_M3_CASE(F, 4)(__VA_ARGS__);    \
    case 5: return JAC_M3_CASE(F, 5)(__VA_ARGS__);    \
    default: return hipErrorInvalidValue;             \
    }

template <typename R>
bool march3d_batch_wide(const Geom &g) {
    return sizeof(R) == 4 && m3_wide(g, sizeof(R));
}

template <typename R>
int64_t march3d_batch_items(const Geom &g, int zseg, int depth) {
    if (sizeof(R) == 8) return rows3d_batch_items(g, zseg, depth);
    if (depth < 1 || depth > march3d_max_depth()) return -1;
    int ns, ng;
    m3_shape<R>(g, depth, 1, ns, ng);
    return (int64_t)ns * ng * ((g.n[2] + zseg - 1) / zseg);
}

template <typename R>
hipError_t launch_march3d_batch(const BatchGrid *grids, const int *prefix, int ngrids, bool src,
                                bool wide, int depth, int zseg, int nitems, hipStream_t st) {
    if (sizeof(R) == 8)
        return launch_rows3d_batch(grids, prefix, ngrids, src, depth, zseg, nitems, st);
#define JAC_M3_CASE(F, T) F<T>
    JAC_M3_SWITCH(depth, m3b_launch_t, grids, prefix, ngrids, src, wide, zseg, nitems, st)
#undef JAC_M3_CASE
}

template <typename R>
hipError_t launch_march3d(const Geom &g, const void *uin, void *uout, const void *b, double *res,
                          const M3Plan &pl, hipStream_t st, int depth) {
    if (pl.row) return launch_rows3d<R>(g, uin, uout, b, res, pl, st, depth);
#define JAC_M3_CASE(F, T) F<R, T>
    JAC_M3_SWITCH(depth, m3_launch_t, g, uin, uout, b, res, pl, st)
#undef JAC_M3_CASE
}

#define JAC_M3_DISPATCH(R)                                                                       \
    template bool march3d_plan<R>(const Geom &, int, int, int, size_t, bool, M3Plan *);          \
    template bool march3d_batch_wide<R>(const Geom &);                                           \
    template int64_t march3d_batch_items<R>(const Geom &, int, int);                             \
    template hipError_t launch_march3d_batch<R>(const BatchGrid *, const int *, int, bool, bool, \
                                                int, int, int, hipStream_t);                     \
    template hipError_t launch_march3d<R>(const Geom &, const void *, void *, const void *,      \
                                          double *, const M3Plan &, hipStream_t, int);
JAC_M3_DISPATCH(float)
JAC_M3_DISPATCH(double)

#endif  // JAC_MARCH3D_DEPTH

}  // namespace jac
