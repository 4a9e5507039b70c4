// Access to a lattice's arrays by node: raw buffer loads and stores of one
// storage element, a node's neighbourhood as index parts, the moments a
// two-pass step keeps between its passes.
#pragma once
#include "lbm_device.h"

namespace lbm {

namespace {

constexpr int RSRC_FLAGS = 0x00020000;  // raw dword buffer, gfx9 family

// raw buffer access of one storage element at byte offsets (voff per lane, soff uniform)
template <class S>
__device__ inline S buf_load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff);
template <>
__device__ inline float buf_load<float>(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
template <>
__device__ inline double buf_load<double>(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
    return __hiloint2double(static_cast<int>(v[1]), static_cast<int>(v[0]));
}
template <>
__device__ inline _Float16 buf_load<_Float16>(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    const unsigned short b = __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0);
    return __builtin_bit_cast(_Float16, b);
}
template <>
__device__ inline bf16_t buf_load<bf16_t>(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    bf16_t o;
    o.bits = __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0);
    return o;
}

// Stores carry the non-temporal cache policy (bit 1 of the buffer
// instruction's policy operand): the step never reads back what it writes, so
// the written lines are evicted first and the L2 keeps the pulled planes whose
// halo rows the neighbouring tiles read again (150 -> 144-146 us per FP32
// step on the 256 x 128 x 64 cap; the same policy on the loads costs 179 us).
constexpr int ST_POLICY = 2;
template <class S>
__device__ inline void buf_store(S v, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff);
template <>
__device__ inline void buf_store<float>(float v, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, voff, soff, ST_POLICY);
}
template <>
__device__ inline void buf_store<double>(double v, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    const unsigned long long u = __double_as_longlong(v);
    __attribute__((ext_vector_type(2))) unsigned int w;
    w[0] = static_cast<unsigned int>(u);
    w[1] = static_cast<unsigned int>(u >> 32);
    __builtin_amdgcn_raw_buffer_store_b64(w, r, voff, soff, ST_POLICY);
}
template <>
__device__ inline void buf_store<_Float16>(_Float16 v, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, v), r, voff, soff, ST_POLICY);
}
template <>
__device__ inline void buf_store<bf16_t>(bf16_t v, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    __builtin_amdgcn_raw_buffer_store_b16(v.bits, r, voff, soff, ST_POLICY);
}

__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void *p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), static_cast<short>(0), static_cast<int>(bytes),
                                             RSRC_FLAGS);
}

constexpr int NB = 256;  // nodes per work-group of both passes, in index order

// Moment q of a node between the passes, kept in the node's own elements of
// the destination arrays (which the second pass overwrites after reading
// them): one array per moment, or two (low and high half) in 16-bit storage.
template <class S>
__device__ inline void put_moment(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t fsE, int q,
                                  typename Codec<S>::C v) {
    if constexpr (sizeof(S) == 2) {
        const uint32_t u = __float_as_uint(v);
        __builtin_amdgcn_raw_buffer_store_b16(static_cast<unsigned short>(u), r, voff, (2 * q) * fsE, 0);
        __builtin_amdgcn_raw_buffer_store_b16(static_cast<unsigned short>(u >> 16), r, voff, (2 * q + 1) * fsE, 0);
    } else if constexpr (sizeof(S) == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, voff, q * fsE, 0);
    } else {
        const unsigned long long u = __double_as_longlong(v);
        __attribute__((ext_vector_type(2))) unsigned int w;
        w[0] = static_cast<unsigned int>(u);
        w[1] = static_cast<unsigned int>(u >> 32);
        __builtin_amdgcn_raw_buffer_store_b64(w, r, voff, q * fsE, 0);
    }
}
template <class S>
__device__ inline typename Codec<S>::C get_moment(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t fsE, int q) {
    if constexpr (sizeof(S) == 2) {
        const uint32_t lo = __builtin_amdgcn_raw_buffer_load_b16(r, voff, (2 * q) * fsE, 0);
        const uint32_t hi = __builtin_amdgcn_raw_buffer_load_b16(r, voff, (2 * q + 1) * fsE, 0);
        return __uint_as_float((lo & 0xFFFFu) | (hi << 16));
    } else {
        return buf_load<S>(r, voff, q * fsE);
    }
}

// A node's coordinates and the index parts of its neighbourhood (wrapped in
// periodic directions, clamped in closed ones).
struct NodeNbr {
    uint32_t xs[3], ys[3], zs[3];
    int z;
    __device__ inline uint32_t at(int dx, int dy, int dz) const { return zs[1 + dz] + ys[1 + dy] + xs[1 + dx]; }
};
template <class Args>
__device__ inline NodeNbr node_nbr(uint32_t n, const Args &a) {
    const uint32_t nx = a.nx, ny = a.ny, nxy = nx * ny;
    const uint32_t z = n / nxy, rem = n - z * nxy, y = rem / nx, x = rem - y * nx;
    NodeNbr o;
    o.z = int(z);
    o.xs[1] = x;
    o.xs[0] = x > 0 ? x - 1 : (a.px ? nx - 1 : 0);
    o.xs[2] = x + 1 < nx ? x + 1 : (a.px ? 0 : x);
    o.ys[1] = y * nx;
    o.ys[0] = y > 0 ? (y - 1) * nx : (a.py ? (ny - 1) * nx : 0);
    o.ys[2] = y + 1 < ny ? (y + 1) * nx : (a.py ? 0 : y * nx);
    o.zs[1] = z * nxy;
    o.zs[0] = z > 0 ? (z - 1) * nxy : (a.pz ? (a.nz - 1) * nxy : 0);
    o.zs[2] = int(z) + 1 < a.nz ? (z + 1) * nxy : (a.pz ? 0 : z * nxy);
    return o;
}

// Work-groups are dealt to the eight XCDs round-robin: each XCD takes a
// contiguous range of nodes, so that the lines two neighbouring work-groups
// share stay in one L2.
__device__ inline int xcd_range(int b, int nblk) { return (nblk & 7) == 0 ? (b & 7) * (nblk >> 3) + (b >> 3) : b; }

}  // namespace

}  // namespace lbm
