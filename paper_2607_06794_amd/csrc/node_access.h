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

// f^eq of one component at a node (Eq. 2) as deviations from w_i rref, in the form
// that every pass shares: with R = rho / 18, A = (rho - rref) / 18 - 3/2 R u^2,
//   f^eq_i - w_i rref = A + R c.u (3 + 9/2 c.u)    (half of it for the diagonals),
// evaluated with the roundings written here and no others, so that a population
// computed again from the same (rho, u) is the same number.  The rest population
// is the remainder, dr - sum of the others, so that sum_i f_i^eq = rho holds up to
// one rounding: the rounded weights do not sum to one, and using them for all 19
// directions would drift the mass by a fixed factor every step.
__device__ inline float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
template <class C>
struct Eq {
    C A, R, u[3];
};
template <class C>
__device__ inline Eq<C> make_eq(C dr, C rho, C ux, C uy, C uz) {
#pragma clang fp contract(off)
    Eq<C> e;
    const C usq = fma_(uz, uz, fma_(uy, uy, ux * ux));
    e.R = wgt<C>(1) * rho;
    e.A = fma_(e.R, C(-1.5) * usq, wgt<C>(1) * dr);
    e.u[0] = ux;
    e.u[1] = uy;
    e.u[2] = uz;
    return e;
}
// c_i . u; u(d): component d of the velocity
template <class C, class F>
__device__ inline C along(int i, F u) {
#pragma clang fp contract(off)
    C cu = C(0);
    if (cx(i)) cu = cx(i) > 0 ? u(0) : -u(0);
    if (cy(i)) cu = cx(i) ? (cy(i) > 0 ? cu + u(1) : cu - u(1)) : (cy(i) > 0 ? u(1) : -u(1));
    if (cz(i)) cu = cx(i) || cy(i) ? (cz(i) > 0 ? cu + u(2) : cu - u(2)) : (cz(i) > 0 ? u(2) : -u(2));
    return cu;
}
// direction i > 0, without the diagonals' half
template <class C, class F>
__device__ inline C eq_pop_full(int i, C A, C R, F u) {
#pragma clang fp contract(off)
    const C cu = along<C>(i, u);
    return fma_(R, cu * fma_(C(4.5), cu, C(3)), A);
}
template <class C>
__device__ inline C eq_pop_full(int i, const Eq<C> &e) {
    return eq_pop_full(i, e.A, e.R, [&](int d) { return e.u[d]; });
}
template <class C>
__device__ inline C eq_pop(int i, const Eq<C> &e) {
    const C f = eq_pop_full(i, e);
    return i <= 6 ? f : C(0.5) * f;
}

// The same populations (i > 0) by opposite pairs, w_i dr + w_i rho (9/2 (c.u)^2 -
// 3/2 u^2) +- w_i rho 3 c.u: the form for 16-bit storage, whose steps never pass on
// moments.  There the last bit of this sum can decide which 16-bit neighbour is
// stored, and the steps after it carry that on (with the form above 2e-4 of the
// populations within 20 steps): these roundings, and the order of u^2, are the ones
// of the one-pass step, so that its runs are repeated bit for bit.  It also takes
// less time than the form above beside the rounding: 20 FP16 steps of 256 x 128 x
// 64 2 060 -> 2 000 us.
template <class C>
__device__ inline void eq_pairs(C dr, C rho, const C (&u)[3], C (&f)[Q]) {
#pragma clang fp contract(off)
    const C base = C(-1.5) * fma_(u[2], u[2], fma_(u[0], u[0], u[1] * u[1]));
#pragma unroll
    for (int i = 1; i < Q; i += 2) {
        const C cu = along<C>(i, [&](int d) { return u[d]; }), wr = wgt<C>(i) * rho, odd = C(3) * cu;
        const C even = fma_(wr, fma_(C(4.5) * cu, cu, base), wgt<C>(i) * dr);
        f[i] = fma_(wr, odd, even);
        f[i + 1] = fma_(-wr, odd, even);
    }
}

// Between the steps of one call with tau = 1 a node is its moments per component
// k: (rho_k - rref_k, u_k^eq) as one vector, element n at 4 (k fs + n), and the
// rest population at (8 + k) fs + n; the others are f^eq_i(rho_k, u_k^eq).
template <class S>
__device__ inline void load_state(__amdgpu_buffer_rsrc_t r, uint32_t n, uint32_t fsE, int k, S (&m)[4]) {
    const uint32_t voff = n * uint32_t(4 * sizeof(S)), soff = uint32_t(4 * k) * fsE;
#pragma unroll
    for (int h = 0; h < int(sizeof(S)) / 4; ++h) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, voff + 16 * h, soff, 0);
        if constexpr (sizeof(S) == 4) {
#pragma unroll
            for (int q = 0; q < 4; ++q) m[q] = __uint_as_float(v[q]);
        } else {
#pragma unroll
            for (int q = 0; q < 2; ++q)
                m[2 * h + q] = __hiloint2double(static_cast<int>(v[2 * q + 1]), static_cast<int>(v[2 * q]));
        }
    }
}
// The store's whole offset is in the lane register: with an SGPR offset the
// compiler lets the next instruction overwrite the data registers of a 16-byte
// store, and lanes were seen to store what it wrote (it keeps the wait state that
// such a store needs only where the offset is a constant).
template <class S>
__device__ inline void store_state(__amdgpu_buffer_rsrc_t r, uint32_t n, uint32_t fsE, int k, const S (&m)[4]) {
    const uint32_t voff = n * uint32_t(4 * sizeof(S)) + uint32_t(4 * k) * fsE;
#pragma unroll
    for (int h = 0; h < int(sizeof(S)) / 4; ++h) {
        __attribute__((ext_vector_type(4))) unsigned int v;
        if constexpr (sizeof(S) == 4) {
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = __float_as_uint(m[q]);
        } else {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const unsigned long long u = __double_as_longlong(m[2 * h + q]);
                v[2 * q] = static_cast<unsigned int>(u);
                v[2 * q + 1] = static_cast<unsigned int>(u >> 32);
            }
        }
        __builtin_amdgcn_raw_buffer_store_b128(v, r, voff + 16 * h, 0, 0);
    }
}
// The entry of a node whose populations are elements of the other population
// buffer (rod nodes: the slots that the link pass wrote; nodes that the update
// pass refilled): a quiet NaN of its own payload, which no arithmetic here
// makes, in place of rho_A - rref_A.
__device__ inline float pop_mark(float) { return __uint_as_float(0x7FC0B0D5u); }
__device__ inline double pop_mark(double) { return __longlong_as_double(0x7FF80B0D50000000ll); }
__device__ inline bool is_pop_mark(float v) { return __float_as_uint(v) == 0x7FC0B0D5u; }
__device__ inline bool is_pop_mark(double v) { return __double_as_longlong(v) == 0x7FF80B0D50000000ll; }

// A node's coordinates and the index parts of its neighbourhood (wrapped in
// periodic directions, clamped in closed ones).
struct NodeNbr {
    uint32_t xs[3], ys[3], zs[3];
    int z;
    __device__ inline uint32_t at(int dx, int dy, int dz) const { return zs[1 + dz] + ys[1 + dy] + xs[1 + dx]; }
};
template <class Args>
__device__ inline NodeNbr node_nbr(uint32_t x, uint32_t y, uint32_t z, const Args &a) {
    const uint32_t nx = a.nx, ny = a.ny, nz = a.nz, nxy = nx * ny;
    NodeNbr o;
    o.z = int(z);
    o.xs[1] = x;
    o.xs[0] = x > 0 ? x - 1 : (a.px ? nx - 1 : 0);
    o.xs[2] = x + 1 < nx ? x + 1 : (a.px ? 0 : x);
    o.ys[1] = y * nx;
    o.ys[0] = y > 0 ? o.ys[1] - nx : (a.py ? (ny - 1) * nx : 0);
    o.ys[2] = y + 1 < ny ? o.ys[1] + nx : (a.py ? 0 : o.ys[1]);
    o.zs[1] = z * nxy;
    o.zs[0] = z > 0 ? o.zs[1] - nxy : (a.pz ? (nz - 1) * nxy : 0);
    o.zs[2] = z + 1 < nz ? o.zs[1] + nxy : (a.pz ? 0 : o.zs[1]);
    return o;
}
template <class Args>
__device__ inline NodeNbr node_nbr(uint32_t n, const Args &a) {
    const uint32_t row = a.by_nx(n), z = a.by_ny(row);
    return node_nbr(n - row * a.nx, row - z * a.ny, z, a);
}

// Work-groups are dealt to the eight XCDs round-robin: each XCD takes a
// contiguous range of nodes, so that the lines two neighbouring work-groups
// share stay in one L2.
__device__ inline int xcd_range(int b, int nblk) { return (nblk & 7) == 0 ? (b & 7) * (nblk >> 3) + (b >> 3) : b; }

}  // namespace

}  // namespace lbm
