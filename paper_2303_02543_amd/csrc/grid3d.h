// Offsets of 3D grid nodes, shared by the 3D pass kernels.
#pragma once

#include "jacobi_internal.h"

namespace jac {

// Element offset of the z part (block layer and plane) of a global plane z.
__device__ __forceinline__ int64_t plane_part(const Geom &g, int zblk, int zloc) {
    return (int64_t)zblk * g.nb[1] * g.nb[0] * g.bstride + (int64_t)(zloc + 1) * g.plane;
}
__device__ __forceinline__ int64_t src_plane_part(const Geom &g, int zblk, int zloc) {
    return (int64_t)zblk * g.nb[1] * g.nb[0] * g.sstride + (int64_t)zloc * g.e[1] * g.e[0];
}
// Element offset of the x/y part of node (x, y) inside its z layer: its
// block column / row and its place in the block's plane (state buffers).
__device__ __forceinline__ int64_t xy_part(const Geom &g, int x, int y) {
    int bx, lx, by, ly;
    owner(x, g.e[0], g.nb[0], bx, lx);
    owner(y, g.e[1], g.nb[1], by, ly);
    return ((int64_t)by * g.nb[0] + bx) * g.bstride + (int64_t)(ly + 1) * g.pitch + g.ax + lx;
}
__device__ __forceinline__ int64_t src_xy_part(const Geom &g, int x, int y) {
    int bx, lx, by, ly;
    owner(x, g.e[0], g.nb[0], bx, lx);
    owner(y, g.e[1], g.nb[1], by, ly);
    return ((int64_t)by * g.nb[0] + bx) * g.sstride + (int64_t)ly * g.e[0] + lx;
}

}  // namespace jac
