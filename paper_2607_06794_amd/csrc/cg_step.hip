// Colour-gradient D3Q19 step for gfx950 (the paper's fluid model; Methods,
// "Fluid-filament simulation method"): per component BGK towards the
// equilibrium of the common velocity (Eqs. 1-3), the capillary force of a
// continuum-surface formulation from the curvature of the colour field
// C = (rho_1 - rho_2) / (rho_1 + rho_2), weighted by the density fractions and
// applied before the collision (Guo's forcing), then recolouring; wetting by
// a ghost colour in the solid layer and wall normals from the voxel geometry,
// the interface normal turned to the wall's contact angle.
//
// The curvature needs the colour two nodes out, so the step runs as passes
// over SoA arrays (thread per node, x fastest, coalesced):
//   1. stream:  pull the 38 populations of each fluid node, C into an array;
//               with tau = 1 also rho_k and j, since the collision then needs
//               nothing else of them (f* = f^eq plus the force);
//   2. ghost:   each static wall node's ghost colour, the w-weighted mean C
//               of its fluid neighbours, into the same array, 0 elsewhere;
//   3. normal:  grad C from the neighbours' C, unit normal with the
//               contact-angle correction next to walls, n and |grad C| into
//               four arrays;
//   4. collide: the moments (tau != 1: pulled and summed again), curvature
//               from the neighbours' normals where the node has a normal,
//               CSF force, Guo-forced BGK per component, recolouring, store,
//               and hand the bounce-back values to the wall nodes.
// Bound by HBM: with tau = 1 the populations are read once and written once
// (pulled twice with tau != 1).  All stencil loads are unconditional (the
// arrays hold neutral values where a neighbour does not count), so that they
// are in flight together.  Per FP32 step of 256 x 128 x 64, before -> now:
//   tau = 1: colour 79, ghost 11, normal 48, collide 168 us -> stream 65,
//   ghost 6.4, normal 12, collide 58 us (4.9 and 5.5 TB/s in the two passes
//   over the populations, a large copy 5.3), 309 -> 141 us with the launches;
//   tau != 1: 309 -> 195 us; FP64: 536 -> 313 and 534 -> 393 us.
#include "lbm_device.h"
#include "lbm_internal.h"
#include "node_access.h"

namespace lbm {

namespace {

// the 38 post-streaming deviations of node neighbourhood nb: f_i(x) =
// f*_i(x - c_i); wall nodes hold the bounce-back values handed to them
template <class S>
__device__ inline void pull(const CGArgs &a, const NodeNbr &nb, typename Codec<S>::C (&fv)[2][Q]) {
    constexpr uint32_t E = sizeof(S);
    const uint32_t fsE = static_cast<uint32_t>(a.fs) * E;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const auto src = make_rsrc(static_cast<const char *>(a.fsrc) + size_t(k) * Q * fsE, Q * fsE);
#pragma unroll
        for (int i = 0; i < Q; ++i)
            fv[k][i] = Codec<S>::dec(buf_load<S>(src, nb.at(-cx(i), -cy(i), -cz(i)) * E, i * fsE));
    }
}

// Eq. 3: rho_k over the populations d_i + w_i rref_k, and j over opposite pairs.
// (Not rref_k + sum_i d_i: where a component is nearly absent its deviations add up
// to -rref_k through partial sums as large, whose rounding is many times that of
// the populations: 6e-8 against 1.4e-8 of rref_k, and a normal nearly along the
// wall's turns that into up to 1e-3 of a population within four steps.)
template <class C>
__device__ inline void moments(const CGArgs &a, const C (&fv)[2][Q], C (&rho)[2], C (&j)[3]) {
#pragma unroll
    for (int d = 0; d < 3; ++d) j[d] = C(0);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        C s = C(0);
#pragma unroll
        for (int i = 0; i < Q; ++i) s += fma_(wgt<C>(i), C(a.rho_ref[k]), fv[k][i]);
        rho[k] = s;
#pragma unroll
        for (int i = 1; i < Q; i += 2) {
            const C d = fv[k][i] - fv[k][i + 1];
            if (cx(i)) j[0] += cx(i) * d;
            if (cy(i)) j[1] += cy(i) * d;
            if (cz(i)) j[2] += cz(i) * d;
        }
    }
}

// ---- pass 1: colour (and, MOM, moments) of every fluid node ----------------
template <class S, bool MOM>
__global__ void __launch_bounds__(NB) cg_stream_kernel(CGArgs a) {
    using C = typename Codec<S>::C;
    const uint32_t n = static_cast<uint32_t>(xcd_range(blockIdx.x, gridDim.x)) * NB + threadIdx.x;
    if (n >= a.nodes) return;
    const bool fluid = (gptr(a.mat)[n] & MAT_ID_MASK) == MAT_FLUID;
    C fv[2][Q], rho[2], j[3];
    pull<S>(a, node_nbr(n, a), fv);
    moments(a, fv, rho, j);
    if (!fluid) return;
    const C rt = rho[0] + rho[1];
    gptr(static_cast<C *>(a.colour))[n] = rt > C(0) ? (rho[0] - rho[1]) / rt : C(0);
    if constexpr (MOM) {
        const uint32_t fsE = static_cast<uint32_t>(a.fs) * sizeof(S);
        const auto dst = make_rsrc(a.fdst, Q * fsE);
#pragma unroll
        for (int d = 0; d < 3; ++d) put_moment<S>(dst, n * sizeof(S), fsE, d, j[d]);
#pragma unroll
        for (int k = 0; k < 2; ++k) put_moment<S>(dst, n * sizeof(S), fsE, 3 + k, rho[k]);
    }
}

// ---- pass 2: ghost colour of the static wall nodes: the w-weighted mean C
// of each wall node's fluid neighbours (0 without any); 0 on other solid nodes.
// So the normal pass reads one value per neighbour and no material.
template <class C>
__global__ void __launch_bounds__(NB) cg_ghost_kernel(CGArgs a) {
    const uint32_t n = static_cast<uint32_t>(xcd_range(blockIdx.x, gridDim.x)) * NB + threadIdx.x;
    if (n >= a.nodes) return;
    const uint8_t m = gptr(a.mat)[n] & MAT_ID_MASK;
    if (m == MAT_FLUID) return;
    auto col = gptr(static_cast<C *>(a.colour));
    if (!is_static_wall(m)) {
        col[n] = C(0);
        return;
    }
    const NodeNbr nb = node_nbr(n, a);
    const int x = int(nb.xs[1]), y = int(a.by_nx(nb.ys[1]));
    const bool in[3][2] = {{a.px || x > 0, a.px || x + 1 < a.nx},
                           {a.py || y > 0, a.py || y + 1 < a.ny},
                           {a.pz || nb.z > 0, a.pz || nb.z + 1 < a.nz}};
    uint8_t mq[Q];
    C cq[Q];
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        const uint32_t q = nb.at(cx(i), cy(i), cz(i));
        mq[i] = gptr(a.mat)[q];
        cq[i] = col[q];
    }
    C num = C(0), den = C(0);
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        bool f = (mq[i] & MAT_ID_MASK) == MAT_FLUID;
        if (cx(i)) f = f && in[0][cx(i) > 0];
        if (cy(i)) f = f && in[1][cy(i) > 0];
        if (cz(i)) f = f && in[2][cz(i) > 0];
        num += f ? wgt<C>(i) * cq[i] : C(0);
        den += f ? wgt<C>(i) : C(0);
    }
    col[n] = den > C(0) ? num / den : C(0);
}

// ---- pass 3: interface normal ---------------------------------------------
template <class C>
__global__ void __launch_bounds__(NB) cg_normal_kernel(CGArgs a) {
    const uint32_t n = static_cast<uint32_t>(xcd_range(blockIdx.x, gridDim.x)) * NB + threadIdx.x;
    if (n >= a.nodes) return;
    const uint8_t mb = gptr(a.mat)[n];
    const NodeNbr nb = node_nbr(n, a);
    const auto col = make_rsrc(a.colour, uint32_t(a.fs) * uint32_t(sizeof(C)));
    // grad C = (1 / c_s^2) sum_i w_i C(x + c_i) c_i, over opposite pairs
    C v[Q];
#pragma unroll
    for (int i = 1; i < Q; ++i) v[i] = buf_load<C>(col, nb.at(cx(i), cy(i), cz(i)) * uint32_t(sizeof(C)), 0);
    C nv[3] = {C(0), C(0), C(0)}, mag = C(0);
    if ((mb & MAT_ID_MASK) == MAT_FLUID) {
        C g[3] = {C(0), C(0), C(0)};
#pragma unroll
        for (int i = 1; i < Q; i += 2) {
            const C d = wgt<C>(i) * (v[i] - v[i + 1]);
            if (cx(i)) g[0] += cx(i) * d;
            if (cy(i)) g[1] += cy(i) * d;
            if (cz(i)) g[2] += cz(i) * d;
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) g[d] *= C(3);
        mag = sqrt(g[0] * g[0] + g[1] * g[1] + g[2] * g[2]);
        if (mag > C(a.grad_eps)) {
#pragma unroll
            for (int d = 0; d < 3; ++d) nv[d] = g[d] / mag;
            if (mb & MAT_NEAR_WALL) {
                // wall normal from the solid neighbours (into the fluid) and
                // their w-weighted mean cos(theta)
                uint8_t mq[Q];
#pragma unroll
                for (int i = 1; i < Q; ++i) mq[i] = gptr(a.mat)[nb.at(cx(i), cy(i), cz(i))] & MAT_ID_MASK;
                C s[3] = {C(0), C(0), C(0)}, ws = C(0), cts = C(0);
#pragma unroll
                for (int i = 1; i < Q; ++i) {
                    if (is_static_wall(mq[i])) {
                        const C w = wgt<C>(i);
                        s[0] += w * C(cx(i));
                        s[1] += w * C(cy(i));
                        s[2] += w * C(cz(i));
                        ws += w;
                        cts += w * C(a.cos_theta[mq[i]]);
                    }
                }
                const C sn = sqrt(s[0] * s[0] + s[1] * s[1] + s[2] * s[2]);
                if (ws > C(0) && sn > C(0)) {
                    const C nw[3] = {-s[0] / sn, -s[1] / sn, -s[2] / sn};
                    const C ct = cts / ws;
                    const C dot = nv[0] * nw[0] + nv[1] * nw[1] + nv[2] * nw[2];
                    C t[3] = {nv[0] - dot * nw[0], nv[1] - dot * nw[1], nv[2] - dot * nw[2]};
                    const C tm = sqrt(t[0] * t[0] + t[1] * t[1] + t[2] * t[2]);
                    if (tm > C(1e-12)) {
                        const C st = sqrt(fmax(C(1) - ct * ct, C(0)));
#pragma unroll
                        for (int d = 0; d < 3; ++d) nv[d] = -ct * nw[d] + st * (t[d] / tm);
                    }
                }
            }
        }
    }
    auto nrm = gptr(static_cast<C *>(a.normal));
    nrm[3 * a.fs + n] = mag;
    // read only where |grad C| is above the threshold; whole wavefronts store
    if (__any(mag > C(a.grad_eps))) {
#pragma unroll
        for (int d = 0; d < 3; ++d) nrm[d * a.fs + n] = nv[d];
    }
}

// ---- pass 4: force, collision, recolouring ---------------------------------
template <class S, bool MOM>
__global__ void __launch_bounds__(NB) cg_collide_kernel(CGArgs a) {
    using C = typename Codec<S>::C;
    constexpr uint32_t E = sizeof(S);
    const uint32_t n = static_cast<uint32_t>(xcd_range(blockIdx.x, gridDim.x)) * NB + threadIdx.x;
    if (n >= a.nodes) return;
    const uint8_t mb = gptr(a.mat)[n];
    if ((mb & MAT_ID_MASK) != MAT_FLUID) return;
    const unsigned known = *a.status;  // status bits already raised before this launch
    const NodeNbr nb = node_nbr(n, a);
    const uint32_t fsE = static_cast<uint32_t>(a.fs) * E;
    const auto dst0 = make_rsrc(a.fdst, Q * fsE);
    const auto nrm = make_rsrc(a.normal, 4 * static_cast<uint32_t>(a.fs) * uint32_t(sizeof(C)));
    const uint32_t fsC = static_cast<uint32_t>(a.fs) * uint32_t(sizeof(C));
    auto normal_at = [&](uint32_t q, int d) { return buf_load<C>(nrm, q * uint32_t(sizeof(C)), d * fsC); };
    C fv[2][Q], rho[2], j[3];
    if constexpr (MOM) {
#pragma unroll
        for (int d = 0; d < 3; ++d) j[d] = get_moment<S>(dst0, n * E, fsE, d);
#pragma unroll
        for (int k = 0; k < 2; ++k) rho[k] = get_moment<S>(dst0, n * E, fsE, 3 + k);
    } else {
        pull<S>(a, nb, fv);
        moments(a, fv, rho, j);
    }
    const C mag = normal_at(n, 3), eps = C(a.grad_eps);
    const C rt = rho[0] + rho[1];
    const C irt = rt > C(0) ? C(1) / rt : C(1);
    // CSF force F = (sigma / 2) kappa |grad C| n plus the body force; without a
    // normal (|grad C| at or below the threshold) n is zero and kappa not needed
    C n0[3] = {C(0), C(0), C(0)}, F[3] = {C(0), C(0), C(0)};
    if (!(mag <= eps)) {
        C v[Q][3], mq[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const uint32_t q = nb.at(cx(i), cy(i), cz(i));
            mq[i] = i ? normal_at(q, 3) : mag;
#pragma unroll
            for (int d = 0; d < 3; ++d)
                if (i == 0 || (d == 0 ? cx(i) : d == 1 ? cy(i) : cz(i))) v[i][d] = normal_at(q, d);
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) n0[d] = mag > eps ? v[0][d] : C(0);
        // curvature kappa = -div n; a neighbour without a normal of its own (not
        // fluid, or |grad C| at or below the threshold) enters with this node's
        C div = C(0);
#pragma unroll
        for (int i = 1; i < Q; ++i) {
            const bool def = mq[i] > eps;
            C d = C(0);
            if (cx(i)) d += cx(i) * (def ? v[i][0] : n0[0]);
            if (cy(i)) d += cy(i) * (def ? v[i][1] : n0[1]);
            if (cz(i)) d += cz(i) * (def ? v[i][2] : n0[2]);
            div += wgt<C>(i) * d;
        }
        const C kappa = C(-3) * div;
#pragma unroll
        for (int d = 0; d < 3; ++d) F[d] = C(0.5) * C(a.sigma) * kappa * mag * n0[d];
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) F[d] += rt * C(a.g[d]);
    // common velocity with the half-force shift
    C u[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) u[d] = (j[d] + C(0.5) * F[d]) * irt;
    const C usq = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    {
        unsigned st = 0;
        if (!(rt > C(0))) st |= ST_RHO;
        if (!(usq <= C(0.09))) st |= (usq != usq) ? ST_NAN : ST_SPEED;
        post_status(a.status, known, st);
    }
    const C uF = u[0] * F[0] + u[1] * F[1] + u[2] * F[2];
    // colour-blind post-collision populations: per component BGK towards
    // f^eq(rho_k, u) plus Guo's source with F_k = (rho_k / rho) F, summed:
    //   tot_i = sum_k (1 - om_k) f_ki + ef w_i shape_i + es src_i
    C ef = rt, es = C(0.5) * (rt * irt);
    C keep[2] = {C(0), C(0)};
    if constexpr (!MOM) {
        const C om[2] = {C(a.omega[0]), C(a.omega[1])};
        ef = om[0] * rho[0] + om[1] * rho[1];
        es = ((C(1) - C(0.5) * om[0]) * rho[0] + (C(1) - C(0.5) * om[1]) * rho[1]) * irt;
#pragma unroll
        for (int k = 0; k < 2; ++k) keep[k] = C(1) - om[k];
    }
    C tot[Q];
    const C sym0 = ef * (C(1) - C(1.5) * usq) - es * C(3) * uF;
    tot[0] = wgt<C>(0) * sym0;
#pragma unroll
    for (int i = 1; i < Q; i += 2) {
        const C cu = C(cx(i)) * u[0] + C(cy(i)) * u[1] + C(cz(i)) * u[2];
        const C cF = C(cx(i)) * F[0] + C(cy(i)) * F[1] + C(cz(i)) * F[2];
        const C sym = wgt<C>(i) * (sym0 + cu * (C(4.5) * ef * cu + C(9) * es * cF));
        const C asym = wgt<C>(i) * (C(3) * (ef * cu + es * cF));
        tot[i] = sym + asym;
        tot[i + 1] = sym - asym;
    }
    if constexpr (!MOM) {
#pragma unroll
        for (int i = 0; i < Q; ++i)
#pragma unroll
            for (int k = 0; k < 2; ++k) tot[i] += keep[k] * (fv[k][i] + wgt<C>(i) * C(a.rho_ref[k]));
    }
    // recolouring: proportional share plus +- beta (rho_1 rho_2 / rho) w_i cos phi_i
    const C seg = C(a.beta) * rho[0] * rho[1] * irt;
    const C fr[2] = {rho[0] * irt, rho[1] * irt};
    C sc[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const C cn = C(cx(i)) * n0[0] + C(cy(i)) * n0[1] + C(cz(i)) * n0[2];
        sc[i] = i == 0 ? C(0) : seg * wgt<C>(i) * (i <= 6 ? cn : cn * C(0.70710678118654752440));
    }
    const bool near_wall = (mb & MAT_NEAR_WALL) != 0;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const auto dst = make_rsrc(static_cast<char *>(a.fdst) + size_t(k) * Q * fsE, Q * fsE);
        S e[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const C o = k == 0 ? fr[0] * tot[i] + sc[i] : fr[1] * tot[i] - sc[i];
            e[i] = Codec<S>::enc(o - wgt<C>(i) * C(a.rho_ref[k]));
            buf_store<S>(e[i], dst, n * E, i * fsE);
        }
        if (near_wall) {
            // halfway bounce-back: the wall node x + c_i holds f*_i(x) as
            // direction opp(i) for the next pull
#pragma unroll
            for (int i = 1; i < Q; ++i) {
                const uint32_t q = nb.at(cx(i), cy(i), cz(i));
                if (is_static_wall(gptr(a.mat)[q] & MAT_ID_MASK)) buf_store<S>(e[i], dst, q * E, opp(i) * fsE);
            }
        }
    }
}

template <class S, bool MOM>
static hipError_t launch_cg(const CGArgs &a, hipStream_t s) {
    const dim3 grid(unsigned((a.nodes + NB - 1) / NB + 7) & ~7u), block(NB);
    hipLaunchKernelGGL((cg_stream_kernel<S, MOM>), grid, block, 0, s, a);
    hipLaunchKernelGGL((cg_ghost_kernel<S>), grid, block, 0, s, a);
    hipLaunchKernelGGL((cg_normal_kernel<S>), grid, block, 0, s, a);
    hipLaunchKernelGGL((cg_collide_kernel<S, MOM>), grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_cg_step(int prec, const CGArgs &a, hipStream_t s) {
    // with tau = 1 the collision forgets the streamed populations
    const bool mom = a.omega[0] == 1.0 && a.omega[1] == 1.0;
    switch (prec) {
        case LB_F64:
            return mom ? launch_cg<double, true>(a, s) : launch_cg<double, false>(a, s);
        case LB_F32:
            return mom ? launch_cg<float, true>(a, s) : launch_cg<float, false>(a, s);
        default:
            return hipErrorInvalidValue;
    }
}

}  // namespace lbm
