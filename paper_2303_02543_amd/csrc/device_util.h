// Small device helpers shared by the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace jac {

template <typename R, int V>
struct alignas(16) Chunk {
    R v[V];
};

// Typed access at a byte offset from a (wave-uniform) base pointer, so the
// compiler can use the scalar-base + 32-bit vector-offset addressing form.
template <typename X>
__device__ __forceinline__ const X &at(const void *base, uint32_t byte_off) {
    return *reinterpret_cast<const X *>(reinterpret_cast<const char *>(base) + byte_off);
}
template <typename X>
__device__ __forceinline__ X &at_mut(void *base, uint32_t byte_off) {
    return *reinterpret_cast<X *>(reinterpret_cast<char *>(base) + byte_off);
}

// Load of a 4-, 8- or 16-byte value at a 32-bit byte offset from a
// wave-uniform base, through a buffer descriptor made of the base: a
// scalar base and one vector register, with no vector address arithmetic.
// (Given a pointer plus a zero-extended offset, the compiler hoists the
// extension out of a loop, holds 64-bit offsets and adds them for every
// access.)  The descriptor covers 4 GiB from the base; offsets are in bounds
// by construction.
template <typename X>
__device__ __forceinline__ X buffer_get(const void *base, uint32_t off) {
    static_assert(sizeof(X) == 4 || sizeof(X) == 8 || sizeof(X) == 16, "4, 8 or 16 bytes");
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, -1, 0x00020000);
    X x;
    if constexpr (sizeof(X) == 16) {
        const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
        __builtin_memcpy(&x, &t, 16);
    } else if constexpr (sizeof(X) == 8) {
        const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
        __builtin_memcpy(&x, &t, 8);
    } else {
        const unsigned int t = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
        __builtin_memcpy(&x, &t, 4);
    }
    return x;
}

// 16-byte store at a 32-bit byte offset from a wave-uniform base through a
// buffer descriptor: lanes that have nothing to store pass kNoStore, and
// `on` = false (uniform) drops the whole store, both by the descriptor's
// bounds check.  So the store is issued on every path, and the compiler's
// waits for later loads can count it: a store under a branch is not counted,
// and every wait for a load then also waits for the stores before it.
constexpr uint32_t kBufferBytes = 0xfffff000u;  // offsets stay below this
constexpr uint32_t kNoStore = 0xfffffff0u;
template <bool NT = false, typename X>
__device__ __forceinline__ void buffer_put16(void *base, uint32_t off, bool on, const X &v) {
    static_assert(sizeof(X) == 16, "16-byte stores only");
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    u32x4 t;
    __builtin_memcpy(&t, &v, 16);
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc(base, 0, on ? kBufferBytes : 0u, 0x00020000);
    __builtin_amdgcn_raw_buffer_store_b128(t, r, off, 0, NT ? 2 : 0);
}

// Store of 4, 8 or 16 bytes with the non-temporal hint (the line is not kept in
// the caches on its way to memory).
template <typename X>
__device__ __forceinline__ void store_nt(X *p, const X &v) {
    static_assert(sizeof(X) == 4 || sizeof(X) == 8 || sizeof(X) == 16, "4, 8 or 16 bytes");
    typedef unsigned int u32xn __attribute__((ext_vector_type(sizeof(X) / 4)));
    u32xn t;
    __builtin_memcpy(&t, &v, sizeof(X));
    __builtin_nontemporal_store(t, reinterpret_cast<u32xn *>(p));
}

// Whole-wave lane shifts through DPP (wave_shr:1 / wave_shl:1).  All 64
// lanes must be active.
// shift_up: lane i receives src of lane i-1; lane 0 keeps `old`.
__device__ __forceinline__ float shift_up(float old, float src) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(src),
                                                      0x138, 0xf, 0xf, false));
}
// shift_down: lane i receives src of lane i+1; lane 63 keeps `old`.
__device__ __forceinline__ float shift_down(float old, float src) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(src),
                                                      0x130, 0xf, 0xf, false));
}
__device__ __forceinline__ double shift_up(double old, double src) {
    const long long o = __double_as_longlong(old), s = __double_as_longlong(src);
    const int lo = __builtin_amdgcn_update_dpp((int)o, (int)s, 0x138, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(s >> 32), 0x138, 0xf, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double shift_down(double old, double src) {
    const long long o = __double_as_longlong(old), s = __double_as_longlong(src);
    const int lo = __builtin_amdgcn_update_dpp((int)o, (int)s, 0x130, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(s >> 32), 0x130, 0xf, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Shifts within each 16-lane row of the wave through DPP (row_shr:1 /
// row_shl:1).  All 64 lanes must be active.
// row_shift_up: lane i receives src of lane i-1 of its row; the row's first
// lane keeps `old`.
__device__ __forceinline__ float row_shift_up(float old, float src) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(src),
                                                      0x111, 0xf, 0xf, false));
}
// row_shift_down: lane i receives src of lane i+1 of its row; the row's last
// lane keeps `old`.
__device__ __forceinline__ float row_shift_down(float old, float src) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(src),
                                                      0x101, 0xf, 0xf, false));
}
__device__ __forceinline__ double row_shift_up(double old, double src) {
    const long long o = __double_as_longlong(old), s = __double_as_longlong(src);
    const int lo = __builtin_amdgcn_update_dpp((int)o, (int)s, 0x111, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(s >> 32), 0x111, 0xf, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double row_shift_down(double old, double src) {
    const long long o = __double_as_longlong(old), s = __double_as_longlong(src);
    const int lo = __builtin_amdgcn_update_dpp((int)o, (int)s, 0x101, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(s >> 32), 0x101, 0xf, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Deterministic wave-wide FP64 sum (fixed xor-butterfly order).
__device__ __forceinline__ double wave_sum(double a) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off, 64);
    return a;
}

// Workgroup renumbering for the 8 XCDs (each with its own L2): the hardware
// deals workgroups round-robin, so physical workgroup p runs on XCD p % 8.
// The returned logical numbering gives each XCD one contiguous range, so
// work items with adjacent logical numbers share an L2.
__device__ __forceinline__ int xcd_logical_block(int p, int nblocks) {
    const int q = nblocks >> 3, rem = nblocks & 7;
    const int x = p & 7;
    return x * q + (x < rem ? x : rem) + (p >> 3);
}

}  // namespace jac
