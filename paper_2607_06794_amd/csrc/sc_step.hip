// Shan-Chen D3Q19 step for gfx950: pull stream + boundaries + moments +
// pseudopotential force + velocity shift + BGK collision + store.  With
// tau = 1 in both components the step runs as two passes of one thread per
// node (further down); otherwise it is one fused pass, described next.
//
// Method: lattice Boltzmann equation per component with BGK relaxation
// (Eq. 1), second-order equilibrium (Eq. 2), moments (Eq. 3); the interfacial
// force is applied before collision as a body force (Methods, interfacial
// tension paragraph) -- here the Shan-Chen cross-component pseudopotential
// force entering through the shifted equilibrium velocity.  Wetting uses solid
// ghost pseudo-densities (the paper's solid ghost layer, Methods).
//
// Layout and schedule
// -------------------
// Populations are SoA arrays f[k*19+i][z][y][x] (x fastest).  A work-group
// owns a 64 x TY column tile and marches a chunk of z planes.  For every plane
// it pulls f_i(x) = f*_i(x - c_i) for its TY rows plus a one-node ring around
// them, sums the densities of all (TY+2) x 66 positions into a 4-plane LDS
// ring of pseudo-potentials, and finishes the plane below once the plane above
// is in LDS.  The force needs no density array in HBM: every population is
// read once and written once; the ring re-reads mostly hit L2.
//
// Addressing: all HBM traffic goes through buffer resources (one per
// component).  The plane being marched is the same for the whole work-group,
// so the array index and the z offset form a wave-uniform scalar offset, and
// each thread keeps nine fixed xy offsets (the 3 x 3 neighbourhood of its
// node): a pull costs no vector address arithmetic.
//
// Boundaries inside the same pass:
//  * static walls (halfway bounce-back): a fluid node next to a wall writes
//    f*_j(x) into the wall node's slot of direction opp(j), so the next pull
//    is branch-free;
//  * the reservoir plane z = nz-1: the plane below it takes w_i rho_top_k for
//    the directions pulled from the reservoir and books the outflow of its
//    stored f*(t) towards the reservoir into a per-tile FP64 ledger slot
//    (deterministic: each tile owns its slot);
//  * rod nodes: the slots the next pull reads are written by the rod link
//    kernel; the step stores zero deviations into all of them beforehand, so
//    that waves cut by a rod store whole lines.  On lattices with rods the
//    step also stores every node's densities (compute precision; zero on rod
//    nodes here, the wall's psi after the two passes), which the rod passes read instead of summing 19 populations per
//    surface node in the order of their lists.
//
// Evaporation sink (separate instantiations; FP32 storage, or FP64 with
// tau = 1): after the collision, an interface node (liquid here, a gas fluid node at z + 1) moves
// min(J0 / (K + h / h0), f*_0^A) from A's rest population to B's (Methods,
// evaporation paragraph; Eq. 8).  h, the column's liquid nodes, comes from
// the previous step's per-chunk counts; this step writes its own.
#include <type_traits>

#include "lbm_device.h"
#include "lbm_internal.h"
#include "node_access.h"

namespace lbm {

namespace {

__device__ inline int wrap1(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }
__device__ inline int wrapmod(int v, int n) {
    int r = v % n;
    return r < 0 ? r + n : r;
}

// A node's 3 x 3 xy neighbourhood as element offsets within a plane:
// xy[a][b] = (y + a - 1) * nx + (x + b - 1) with periodic wrap (clamped when
// the direction is closed, where fluid nodes never reach the end planes).
struct NodeXY {
    uint32_t xy[3][3];
    bool valid;
};

__device__ inline NodeXY make_node(int x, int y, const StepArgs &a) {
    NodeXY n;
    bool vx, vy;
    if (a.px) {
        x = wrapmod(x, a.nx);
        vx = true;
    } else {
        vx = (x >= 0 && x < a.nx);
    }
    if (a.py) {
        y = wrapmod(y, a.ny);
        vy = true;
    } else {
        vy = (y >= 0 && y < a.ny);
    }
    n.valid = vx && vy;
    x = min(max(x, 0), a.nx - 1);
    y = min(max(y, 0), a.ny - 1);
    const int xs[3] = {a.px ? wrap1(x - 1, a.nx) : max(x - 1, 0), x, a.px ? wrap1(x + 1, a.nx) : min(x + 1, a.nx - 1)};
    const int ys[3] = {a.py ? wrap1(y - 1, a.ny) : max(y - 1, 0), y, a.py ? wrap1(y + 1, a.ny) : min(y + 1, a.ny - 1)};
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int q = 0; q < 3; ++q) n.xy[p][q] = static_cast<uint32_t>(ys[p]) * a.nx + xs[q];
    return n;
}

template <class C>
__device__ inline C wave_sum(C v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

}  // namespace

// One work-group's tile: logical tile b of a lattice whose step runs as nblk
// work-groups.  remap: b is a hardware dispatch index to be spread over the
// XCDs (else b is already the logical tile).
template <class S, int TY, bool SINK>
__device__ __forceinline__ void sc_step_tile(const StepArgs &a, int b, int nblk, bool remap) {
    using C = typename Codec<S>::C;
    constexpr int TX = 64;
    constexpr int NT = TX * TY;
    constexpr int HX = TX + 2, HY = TY + 2, PL = HX * HY;
    constexpr int NH = 2 * HX + 2 * TY;
    constexpr int NHPT = (NH + NT - 1) / NT;
    constexpr int NW = NT / 64;
    constexpr uint32_t E = sizeof(S);
    __shared__ C ring[4][2][PL];
    __shared__ C psi_tab[16][2];
    __shared__ double red[NW][2];

    // ---- tile of this work-group.  Work-groups are dealt to the eight XCDs
    // round-robin; the remap gives each XCD a contiguous range of logical
    // tiles, ordered z-chunk fastest, so an XCD owns whole xy columns and
    // neighbouring columns (their shared ring reads then hit its L2).
    if (remap && (nblk & 7) == 0) b = (b & 7) * (nblk >> 3) + (b >> 3);
    const int tz = b % a.nzc;
    const int tx = (b / a.nzc) % a.ntx;
    const int ty = b / (a.nzc * a.ntx);
    const int x0 = tx * TX, y0 = ty * TY;
    const int z0 = tz * a.zchunk;
    const int z1 = min(z0 + a.zchunk, a.nz);
    if (z0 >= a.nz) return;  // uniform per block
    // even chunks march up, odd chunks march down: two chunks meet at their
    // shared boundary plane at the same time (both at the start or both at
    // the end of their marches), so the boundary pulls are shared in cache
    const int dir = (tz & 1) ? -1 : 1;
    const int zfirst = dir > 0 ? z0 : z1 - 1;
    const int nplanes = z1 - z0;

    const int tid = threadIdx.x;
    const int lx = tid & 63;
    const int ly = tid >> 6;
    const uint32_t nxy = static_cast<uint32_t>(a.nx) * a.ny;
    const uint32_t fsE = static_cast<uint32_t>(a.fs) * E;  // bytes between population arrays

    // one buffer resource per component over its 19 arrays
    __amdgpu_buffer_rsrc_t src[2], dst[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        src[k] = make_rsrc(static_cast<const char *>(a.fsrc) + size_t(k) * Q * fsE, Q * fsE);
        dst[k] = make_rsrc(static_cast<const char *>(a.fdst) + size_t(k) * Q * fsE, Q * fsE);
    }
    const __amdgpu_buffer_rsrc_t matr = make_rsrc(a.mat, nxy * a.nz);

    if (tid < 32) psi_tab[tid >> 1][tid & 1] = C(a.psi_tab[tid]);
    const unsigned known = *a.status;  // status bits already raised before this launch

    // constants in compute precision; rref is the storage reference density
    // (populations travel as d_i = f_i - w_i rref)
    const C G = C(a.G);
    const C rref[2] = {C(a.rho_ref[0]), C(a.rho_ref[1])};
    const C tdev[2] = {C(a.rho_top[0] - a.rho_ref[0]), C(a.rho_top[1] - a.rho_ref[1])};
    const C om[2] = {C(a.omega[0]), C(a.omega[1])};
    const C ta[2] = {C(a.tau[0]), C(a.tau[1])};
    const C gb[3] = {C(a.g[0]), C(a.g[1]), C(a.g[2])};

    // ---- owned interior node and ring (halo) nodes of this thread
    const NodeXY own = make_node(x0 + lx, y0 + ly, a);
    const bool own_fin = (x0 + lx < a.nx) && (y0 + ly < a.ny);
    const int own_ring = (ly + 1) * HX + (lx + 1);
    NodeXY hal[NHPT];
    int hal_ring[NHPT];
    bool hal_on[NHPT];
#pragma unroll
    for (int m = 0; m < NHPT; ++m) {
        const int h = tid + m * NT;
        int hx = 0, hy = 0;
        hal_on[m] = h < NH;
        if (h < HX) {
            hx = h;
            hy = 0;
        } else if (h < 2 * HX) {
            hx = h - HX;
            hy = HY - 1;
        } else if (h < 2 * HX + TY) {
            hx = 0;
            hy = 1 + h - 2 * HX;
        } else {
            hx = HX - 1;
            hy = 1 + h - 2 * HX - TY;
        }
        if (!hal_on[m]) hx = hy = 0;
        hal[m] = make_node(x0 + hx - 1, y0 + hy - 1, a);
        hal_ring[m] = hy * HX + hx;
    }
    __syncthreads();  // psi_tab

    // evaporation sink (Eq. 8): flux of each owned column from the heights
    // the previous step counted over all z chunks, this chunk's count of
    // liquid nodes after the sink, and the mass this thread moved A -> B
    C sink_J = C(0);
    int sink_cnt = 0;
    double sink_mv = 0.0;
    if constexpr (SINK) {
        int h = 0;
        if (own_fin)
            for (int q = 0; q < a.nzc; ++q) h += a.h_read[size_t(q) * nxy + own.xy[1][1]];
        sink_J = C(a.sink_J0) / (C(a.sink_K) + C(h) / C(a.sink_h0));
    }

    // moments and populations of the owned node: current plane and next plane
    C cur_rho[2], cur_drho[2], cur_j[2][3], cur_f[2][Q];
    C nxt_rho[2], nxt_drho[2], nxt_j[2][3], nxt_f[2][Q];
    uint8_t cur_m, nxt_m;

    // raw pulled values of one plane, in flight between issue() and process()
    S raw_own[2][Q];
    S raw_hal[NHPT][2][Q];
    uint8_t mat_own, mat_hal[NHPT];
    bool plane_valid = false, plane_top = false;

    // psi of a node given its material byte and densities
    auto psi_of = [&](uint8_t m, int k, C rho) -> C {
        const uint8_t id = m & MAT_ID_MASK;
        return id == MAT_FLUID ? rho : psi_tab[id][k];
    };

    // Issue the pulls f*_i(x - c_i) of plane z for the owned and ring nodes.
    // Loads are unconditional (every offset is wrapped or clamped into the
    // lattice); values pulled for non-fluid nodes are discarded by process().
    // Directions pulled from the reservoir plane are not loaded.
    auto issue = [&](int z) {
        int zz = z;
        if (a.pz) {
            zz = wrap1(z, a.nz);
            plane_valid = true;
        } else {
            plane_valid = (z >= 0 && z < a.nz);
        }
        zz = min(max(zz, 0), a.nz - 1);
        const int zm = a.pz ? wrap1(zz - 1, a.nz) : max(zz - 1, 0);
        const int zp = a.pz ? wrap1(zz + 1, a.nz) : min(zz + 1, a.nz - 1);
        const uint32_t zoE[3] = {zm * nxy * E, zz * nxy * E, zp * nxy * E};
        plane_top = a.evap && (zz == a.nz - 2);
        mat_own = uint8_t(__builtin_amdgcn_raw_buffer_load_b8(matr, own.xy[1][1], zz * nxy, 0));
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int i = 0; i < Q; ++i)
                if (!(cz(i) == -1 && plane_top))
                    raw_own[k][i] =
                        buf_load<S>(src[k], own.xy[1 - cy(i)][1 - cx(i)] * E, i * fsE + zoE[1 - cz(i)]);
#pragma unroll
        for (int mm = 0; mm < NHPT; ++mm) {
            if (!hal_on[mm]) continue;
            mat_hal[mm] = uint8_t(__builtin_amdgcn_raw_buffer_load_b8(matr, hal[mm].xy[1][1], zz * nxy, 0));
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int i = 0; i < Q; ++i)
                    if (!(cz(i) == -1 && plane_top))
                        raw_hal[mm][k][i] =
                            buf_load<S>(src[k], hal[mm].xy[1 - cy(i)][1 - cx(i)] * E, i * fsE + zoE[1 - cz(i)]);
        }
    };

    // decoded deviation d_i of a raw pulled value (reservoir sources: w_i (rho_top - rref))
    auto devof = [&](const S (&raw)[2][Q], int k, int i) -> C {
        return (cz(i) == -1 && plane_top) ? wgt<C>(i) * tdev[k] : Codec<S>::dec(raw[k][i]);
    };

    // Turn the issued plane into psi values in ring slot z & 3 and, when
    // keep, into the owned nodes' moments for the next finish.
    auto process = [&](int z, bool keep) {
        const int slot = z & 3;
        const bool v = plane_valid && own.valid;
        const uint8_t m = v ? mat_own : uint8_t(MAT_ID_MASK);
        C rho[2] = {C(0), C(0)}, drho[2] = {C(0), C(0)};
        C j[2][3] = {{C(0), C(0), C(0)}, {C(0), C(0), C(0)}};
        const bool fl = v && (m & MAT_ID_MASK) == MAT_FLUID;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            C fv[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i) fv[i] = devof(raw_own, k, i);
            C s = C(0), jx = C(0), jy = C(0), jz = C(0);
#pragma unroll
            for (int i = 0; i < Q; ++i) s += fv[i];
            // momentum over opposite pairs: f_i - f_opp(i) is nearly exact
            // (the two are close), which avoids cancellation in j
#pragma unroll
            for (int i = 1; i < Q; i += 2) {
                const C d = fv[i] - fv[i + 1];
                if (cx(i) == 1) jx += d;
                if (cx(i) == -1) jx -= d;
                if (cy(i) == 1) jy += d;
                if (cy(i) == -1) jy -= d;
                if (cz(i) == 1) jz += d;
                if (cz(i) == -1) jz -= d;
            }
            // Eq. 3: rho_k = sum_i f_i = rref_k + sum_i d_i (sum_i w_i = 1)
            drho[k] = fl ? s : C(0);
            rho[k] = fl ? rref[k] + s : C(0);
            j[k][0] = fl ? jx : C(0);
            j[k][1] = fl ? jy : C(0);
            j[k][2] = fl ? jz : C(0);
            if (keep) {
#pragma unroll
                for (int i = 0; i < Q; ++i) nxt_f[k][i] = fv[i];
            }
        }
        ring[slot][0][own_ring] = v ? psi_of(m, 0, rho[0]) : C(0);
        ring[slot][1][own_ring] = v ? psi_of(m, 1, rho[1]) : C(0);
        if (keep) {
            nxt_m = m;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                nxt_rho[k] = rho[k];
                nxt_drho[k] = drho[k];
#pragma unroll
                for (int d = 0; d < 3; ++d) nxt_j[k][d] = j[k][d];
            }
        }
#pragma unroll
        for (int mm = 0; mm < NHPT; ++mm) {
            if (!hal_on[mm]) continue;
            const bool v = plane_valid && hal[mm].valid;
            const uint8_t m = v ? mat_hal[mm] : uint8_t(MAT_ID_MASK);
            const bool fl = v && (m & MAT_ID_MASK) == MAT_FLUID;
            C rho[2] = {C(0), C(0)};
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                C s = C(0);
#pragma unroll
                for (int i = 0; i < Q; ++i) s += devof(raw_hal[mm], k, i);
                rho[k] = fl ? rref[k] + s : C(0);
            }
            ring[slot][0][hal_ring[mm]] = v ? psi_of(m, 0, rho[0]) : C(0);
            ring[slot][1][hal_ring[mm]] = v ? psi_of(m, 1, rho[1]) : C(0);
        }
    };

    auto shift_next = [&]() {
        cur_m = nxt_m;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            cur_rho[k] = nxt_rho[k];
            cur_drho[k] = nxt_drho[k];
#pragma unroll
            for (int d = 0; d < 3; ++d) cur_j[k][d] = nxt_j[k][d];
#pragma unroll
            for (int i = 0; i < Q; ++i) cur_f[k][i] = nxt_f[k][i];
        }
    };

    // prologue: the plane behind the first one (psi only), the first plane
    // (psi, moments and populations)
    issue(zfirst - dir);
    process(zfirst - dir, false);
    issue(zfirst);
    process(zfirst, true);
    shift_next();

    for (int it = 0; it < nplanes; ++it) {
        const int z = zfirst + it * dir;
        // the ring holds 4 planes: this iteration writes plane z + dir and
        // reads z - 1, z, z + 1; the next one writes z + 2 dir, which no
        // thread of this iteration reads, so one barrier per plane suffices
        issue(z + dir);
        process(z + dir, true);
        __syncthreads();

        const int sm = (z - 1) & 3, s0 = z & 3, sp = (z + 1) & 3;
        const uint32_t zE = static_cast<uint32_t>(z) * nxy * E;
        const bool ledger_plane = a.evap && (z == a.nz - 2);
        double led[2] = {0.0, 0.0};
        unsigned st = 0;

        // rod nodes go through the same arithmetic (all their moments are
        // zero, so every deviation they store is exactly zero) and store
        // with the fluid lanes: a wave that a rod cuts through then still
        // writes whole lines, where masked lanes would leave partial lines
        // that HBM has to read, merge and write back.  Nothing reads these
        // slots before the rod passes rewrite them (link) or refill them.
        const uint8_t mid = cur_m & MAT_ID_MASK;
        if (own_fin && (mid == MAT_FLUID || mid == MAT_ROD)) {
            const bool fluid = mid == MAT_FLUID;
            const int rc = own_ring;
            const C rho[2] = {cur_rho[0], cur_rho[1]};
            if (a.rho_out) {  // lattices with rods: the densities for the rod passes
                C *ro = static_cast<C *>(a.rho_out);
                const int64_t nn = int64_t(z) * nxy + own.xy[1][1];
                ro[nn] = rho[0];
                ro[a.fs + nn] = rho[1];
            }
            // interface node of the sink: liquid here (rho_A > rho_B) and a
            // gas fluid node above, whose densities are its psi in the ring
            bool sink_if = false;
            C sink_d = C(0);
            if constexpr (SINK) {
                if (rho[0] > rho[1] && (a.pz || z + 1 < a.nz) && ring[sp][0][rc] < ring[sp][1][rc]) {
                    const int za = a.pz ? wrap1(z + 1, a.nz) : z + 1;
                    const uint8_t ma = uint8_t(__builtin_amdgcn_raw_buffer_load_b8(matr, own.xy[1][1], za * nxy, 0));
                    sink_if = (ma & MAT_ID_MASK) == MAT_FLUID;
                }
            }
            // Shan-Chen force: F_k = -G psi_k(x) sum_i w_i psi_kbar(x + c_i) c_i + rho_k g
            C F[2][3];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int kb = 1 - k;
                // sum_i w_i psi(x + c_i) c_i taken over opposite pairs as central
                // differences w_i c_i (psi(x + c_i) - psi(x - c_i)): no cancellation
                C sx = C(0), sy = C(0), sz = C(0);
#pragma unroll
                for (int i = 1; i < Q; i += 2) {
                    const int slp = cz(i) == 1 ? sp : (cz(i) == -1 ? sm : s0);
                    const int slm = cz(i) == 1 ? sm : (cz(i) == -1 ? sp : s0);
                    const C nb = wgt<C>(i) * (ring[slp][kb][rc + cy(i) * HX + cx(i)] -
                                              ring[slm][kb][rc - cy(i) * HX - cx(i)]);
                    if (cx(i) == 1) sx += nb;
                    if (cx(i) == -1) sx -= nb;
                    if (cy(i) == 1) sy += nb;
                    if (cy(i) == -1) sy -= nb;
                    if (cz(i) == 1) sz += nb;
                    if (cz(i) == -1) sz -= nb;
                }
                const C gp = -G * rho[k];
                F[k][0] = gp * sx + rho[k] * gb[0];
                F[k][1] = gp * sy + rho[k] * gb[1];
                F[k][2] = gp * sz + rho[k] * gb[2];
            }
            // velocity shift: u' = sum_k j_k/tau_k / sum_k rho_k/tau_k; u_k^eq = u' + tau_k F_k / rho_k
            const C den = rho[0] * om[0] + rho[1] * om[1];
            const C rden = den > C(0) ? C(1) / den : C(0);
            C up[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) up[d] = (cur_j[0][d] * om[0] + cur_j[1][d] * om[1]) * rden;
            // health check on the physical velocity (sum_k j_k + F/2) / rho
            {
                const C rt = rho[0] + rho[1];
                const C ir = rt > C(0) ? C(1) / rt : C(0);
                C usq_chk = C(0);
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const C ud = (cur_j[0][d] + cur_j[1][d] + C(0.5) * (F[0][d] + F[1][d])) * ir;
                    usq_chk += ud * ud;
                }
                if (fluid && !(rt > C(0))) st |= ST_RHO;
                if (fluid && !(usq_chk <= C(0.09))) st |= (usq_chk != usq_chk) ? ST_NAN : ST_SPEED;
            }

            const uint32_t voE = own.xy[1][1] * E;
            const bool near_wall = fluid && (cur_m & MAT_NEAR_WALL) != 0;
            // 16-bit storage with stochastic rounding: the random bits depend on
            // (node, array, step) only; the wall slots reuse the encoded values
            const int64_t gnode = int64_t(z) * nxy + own.xy[1][1];
            SrStream sr{0u, 0u};
            if constexpr (sizeof(S) == 2) {
                if (a.sr_key) sr.state = sr_seed(a.sr_key, gnode);
            }
            auto encode = [&](C v, int arr) -> S {
                if constexpr (sizeof(S) == 2) {
                    if (a.sr_key) return Stochastic<S>::enc(v, sr.bits(arr));
                }
                return Codec<S>::enc(v);
            };
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                C ue[3];
                const bool ok = rho[k] >= C(1e-12);
                const C rk = ok ? ta[k] / rho[k] : C(0);
#pragma unroll
                for (int d = 0; d < 3; ++d) ue[d] = up[d] + F[k][d] * rk;
                const C usq = ue[0] * ue[0] + ue[1] * ue[1] + ue[2] * ue[2];
                const C dr = cur_drho[k];
                S sstar[Q];
                C deq_sum = C(0);
                // Eq. 2 as a deviation, built per opposite pair (i, opp(i)):
                //   f^eq - w rref = w (rho - rref) + w rho [9/2 (c.u)^2 - 3/2 u^2]  +-  w rho 3 c.u
                // The rest population is the remainder so that sum_i f_i^eq = rho holds up to
                // one rounding: the rounded weights do not sum to one, and using them for all
                // 19 directions would drift the mass by a fixed factor every step.
                C deq[Q];
                const C base = C(-1.5) * usq;
#pragma unroll
                for (int i = 1; i < Q; i += 2) {
                    const C cu = C(cx(i)) * ue[0] + C(cy(i)) * ue[1] + C(cz(i)) * ue[2];
                    const C wr = wgt<C>(i) * rho[k];
                    const C sym = wgt<C>(i) * dr + wr * (base + C(4.5) * cu * cu);
                    const C asym = wr * (C(3) * cu);
                    deq[i] = sym + asym;
                    deq[i + 1] = sym - asym;
                    deq_sum += deq[i];
                    deq_sum += deq[i + 1];
                }
                deq[0] = dr - deq_sum;
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    C ds = fluid ? cur_f[k][i] - (cur_f[k][i] - deq[i]) * om[k] : C(0);
                    if constexpr (SINK) {
                        // Eq. 8: min(J, f*_0^A), at least 0, leaves A's rest population for B's
                        if (i == 0 && sink_if) {
                            if (k == 0) {
                                sink_d = fmax(fmin(sink_J, ds + wgt<C>(0) * rref[0]), C(0));
                                ds -= sink_d;
                            } else {
                                ds += sink_d;
                            }
                        }
                    }
                    sstar[i] = encode(ds, k * Q + i);
                    buf_store<S>(sstar[i], dst[k], voE, i * fsE + zE);
                }
                if (ledger_plane && fluid) {
                    // this step's streaming moves the node's stored f*_i(t) with c_iz = +1
                    // into the reservoir and pulls w_i rho_top_k out of it
                    double outflow = 0.0, inflow = 0.0;
#pragma unroll
                    for (int i = 0; i < Q; ++i) {
                        if (cz(i) == 1)
                            outflow += double(Codec<S>::dec(buf_load<S>(src[k], voE, i * fsE + zE))) +
                                       wgt<double>(i) * a.rho_ref[k];
                        if (cz(i) == -1) inflow += wgt<double>(i) * a.rho_top[k];
                    }
                    led[k] += outflow - inflow;
                }
                if (near_wall) {
                    // halfway bounce-back: hand f*_j(x) to the wall node x + c_j as
                    // direction opp(j) (w_j = w_opp(j), so the deviation carries over)
                    const uint32_t zl[3] = {
                        static_cast<uint32_t>(a.pz ? wrap1(z - 1, a.nz) : max(z - 1, 0)) * nxy,
                        static_cast<uint32_t>(z) * nxy,
                        static_cast<uint32_t>(a.pz ? wrap1(z + 1, a.nz) : min(z + 1, a.nz - 1)) * nxy};
#pragma unroll
                    for (int jd = 1; jd < Q; ++jd) {
                        const uint32_t nxyo = own.xy[1 + cy(jd)][1 + cx(jd)];
                        const uint8_t nm = uint8_t(__builtin_amdgcn_raw_buffer_load_b8(matr, nxyo, zl[1 + cz(jd)], 0));
                        if (is_static_wall(nm & MAT_ID_MASK))
                            buf_store<S>(sstar[jd], dst[k], nxyo * E,
                                         opp(jd) * fsE + zl[1 + cz(jd)] * E);
                    }
                }
            }
            if constexpr (SINK) {
                // the column height the next step reads: liquid after the sink
                sink_cnt += (rho[0] - sink_d > rho[1] + sink_d) ? 1 : 0;
                sink_mv += double(sink_d);
            }
        }
        post_status(a.status, known, st);

        if (ledger_plane) {  // uniform across the block
            const int w = tid >> 6;
            double l0 = wave_sum(led[0]), l1 = wave_sum(led[1]);
            if (lx == 0) {
                red[w][0] = l0;
                red[w][1] = l1;
            }
            __syncthreads();
            if (tid == 0) {
                double s0v = 0.0, s1v = 0.0;
                for (int q = 0; q < NW; ++q) {
                    s0v += red[q][0];
                    s1v += red[q][1];
                }
                double *slot = a.ledger_part + 2 * (ty * a.ntx + tx);
                slot[0] += s0v;
                slot[1] += s1v;
            }
        }
        shift_next();
    }

    if constexpr (SINK) {
        // this chunk's column heights, and the work-group's moved mass into
        // its own ledger pair (A loses it, B gains it)
        if (own_fin) a.h_write[size_t(tz) * nxy + own.xy[1][1]] = sink_cnt;
        const double mv = wave_sum(sink_mv);
        __syncthreads();  // red may still be read by the last ledger plane's sum
        if (lx == 0) red[tid >> 6][0] = mv;
        __syncthreads();
        if (tid == 0) {
            double sum = 0.0;
            for (int q = 0; q < NW; ++q) sum += red[q][0];
            double *slot = a.sink_ledger + 2 * ((size_t(tz) * a.nty + ty) * a.ntx + tx);
            slot[0] += sum;
            slot[1] -= sum;
        }
    }
}

template <class S, int TY, bool SINK>
__global__ void __launch_bounds__(64 * TY) sc_step_kernel(StepArgs a) {
    sc_step_tile<S, TY, SINK>(a, blockIdx.x, gridDim.x, true);
}

// Batched step: one launch walks a device work list of (lattice, logical
// tile) entries over many lattices of one tile class, each with its own
// parameter record.  The list is ordered so that the hardware's round-robin
// dealing of work-groups to XCDs gives each XCD a contiguous range of it.
template <class S, int TY>
__global__ void __launch_bounds__(64 * TY) sc_step_batch_kernel(const StepArgs *__restrict__ all,
                                                                const int2 *__restrict__ work) {
    const int2 w = work[blockIdx.x];
    if (w.x < 0) return;  // padding entry, uniform per block
    const StepArgs a = all[w.x];
    sc_step_tile<S, TY, false>(a, w.y, a.ntx * a.nty * a.nzc, false);
}

// ---------------------------------------------------------------------------
// The step in two passes (tau = 1).  The collision with tau = 1
// forgets the streamed populations, f* = f^eq(rho_k, u_k^eq), so a node needs
// only its moments: the stream pass pulls the 38 populations and keeps psi_k
// (an array of its own, read with its neighbours by the second pass) and
// j = j_A + j_B; the collide pass forms the force, the shifted velocities and
// stores the 38 equilibria.
//
// Both passes are bound by HBM: 152 + 20 bytes read or written per FP32 node
// each (the 20 come back from the caches).  The fused pass pulls the ring of
// its tile again (1.22 x the reads), keeps two waves per SIMD (211 VGPRs) and
// marches z in series, so a small lattice filled a few CUs only.  Measured per
// step, fused -> two passes (stream + collide):
//   FP32 256 x 128 x 64: 145 -> 120 us (5.3 TB/s, the rate of a large copy);
//     with the densities of a rod lattice stored, 162 -> 134 us
//   FP16, stochastic: 137 -> 80 us;  FP64: 299 us (5.1 TB/s)
//   FP32 117 x 51 x 37: 61 -> 18 us;  FP64 32^3: 64 -> 10.5 us (two launches)
// so tau = 1 always takes this form.  With tau != 1 the collision needs the
// populations themselves, which would have to be pulled or stored once more.
//
// The stores of the populations are non-temporal: plain ones take 154 us per
// FP32 step (they evict the lines of the next pull).  The blocks of the stream
// pass in reverse order, to find the last stores in the memory-side cache:
// 125 us.
// ---------------------------------------------------------------------------
__host__ __device__ int split_blocks(int nx, int ny, int nz) { return int((int64_t(nx) * ny * nz + NB - 1) / NB); }

// Books one streaming's exchange with the reservoir into the slot of block b:
// out(k, i) = f*_i - w_i rref_k of a node below it (here), for c_iz = +1.
template <class F>
__device__ __forceinline__ void book_top(const StepArgs &a, int b, bool here, double (&red)[NB / 64][2], F out) {
    const uint32_t nxy = static_cast<uint32_t>(a.nx) * a.ny;
    const uint32_t b0 = a.evap ? (uint32_t(a.nz - 2) * nxy) / NB : 0;
    if (!(a.evap && uint32_t(b) >= b0 && uint32_t(b) <= (uint32_t(a.nz - 1) * nxy - 1) / NB)) return;  // uniform
    double led[2] = {0.0, 0.0};
    if (here) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            double outflow = 0.0, inflow = 0.0;
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                if (cz(i) == 1) outflow += double(out(k, i)) + wgt<double>(i) * a.rho_ref[k];
                if (cz(i) == -1) inflow += wgt<double>(i) * a.rho_top[k];
            }
            led[k] = outflow - inflow;
        }
    }
    const double l0 = wave_sum(led[0]), l1 = wave_sum(led[1]);
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6][0] = l0;
        red[threadIdx.x >> 6][1] = l1;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double s = 0.0;
        for (int q = 0; q < NB / 64; ++q) s += red[q][threadIdx.x];
        a.ledger_part[2 * (b - b0) + threadIdx.x] += s;
    }
}

// Sums of component k's streamed deviations fv (Eq. 3): rho_k - rref_k and j_k.
// top: the plane below the reservoir, which sends w_i rho_top_k.  FULL: fv holds
// twice the diagonals' deviations; halving is exact, so the sums are the same.
template <bool FULL = false, class C>
__device__ __forceinline__ void stream_moments(const StepArgs &a, int k, bool top, C (&fv)[Q], C &dr, C (&j)[3]) {
    const C tdev = C(a.rho_top[k] - a.rho_ref[k]);
#pragma unroll
    for (int i = 0; i < Q; ++i)
        if (cz(i) == -1) fv[i] = top ? wgt<C>(FULL ? 1 : i) * tdev : fv[i];
    auto add = [](C s, C v, int i) { return FULL && i > 6 ? fma_(C(0.5), v, s) : s + v; };
    C s = C(0), jx = C(0), jy = C(0), jz = C(0);
#pragma unroll
    for (int i = 0; i < Q; ++i) s = add(s, fv[i], i);
    // momentum over opposite pairs: f_i - f_opp(i) is nearly exact
    // (the two are close), which avoids cancellation in j
#pragma unroll
    for (int i = 1; i < Q; i += 2) {
        const C d = fv[i] - fv[i + 1];
        if (cx(i)) jx = add(jx, cx(i) > 0 ? d : -d, i);
        if (cy(i)) jy = add(jy, cy(i) > 0 ? d : -d, i);
        if (cz(i)) jz = add(jz, cz(i) > 0 ? d : -d, i);
    }
    dr = s;
    j[0] = jx;
    j[1] = jy;
    j[2] = jz;
}

// Node n after streaming: psi_k into a.rho_out, j (and, with a storage
// reference, the deviations) into a.jm.
template <class S>
__device__ __forceinline__ void stream_store(const StepArgs &a, uint32_t n, uint8_t m, const typename Codec<S>::C (&dr)[2],
                                             const typename Codec<S>::C (&j)[2][3]) {
    using C = typename Codec<S>::C;
    constexpr uint32_t E = sizeof(S);
    const uint32_t fsE = static_cast<uint32_t>(a.fs) * E;
    const bool fluid = m == MAT_FLUID;
    // sum_i f_i = rref_k + sum_i d_i (sum_i w_i = 1)
    C rho[2] = {C(a.rho_ref[0]) + dr[0], C(a.rho_ref[1]) + dr[1]};
    C *psi = static_cast<C *>(a.rho_out);
    if (!fluid) {
        rho[0] = C(gptr(a.psi_tab)[2 * m]);
        rho[1] = C(gptr(a.psi_tab)[2 * m + 1]);
    }
    gptr(psi)[n] = rho[0];
    gptr(psi)[a.fs + n] = rho[1];
    if (fluid) {
        const auto dst = make_rsrc(a.jm, Q * fsE);
#pragma unroll
        for (int d = 0; d < 3; ++d) put_moment<S>(dst, n * E, fsE, d, j[0][d] + j[1][d]);
        if (a.rho_ref[0] != 0.0 || a.rho_ref[1] != 0.0) {
            put_moment<S>(dst, n * E, fsE, 3, dr[0]);
            put_moment<S>(dst, n * E, fsE, 4, dr[1]);
        }
    }
}

template <class S>
__device__ __forceinline__ void sc_stream_nodes(const StepArgs &a, int b) {
    using C = typename Codec<S>::C;
    constexpr uint32_t E = sizeof(S);
    __shared__ double red[NB / 64][2];
    const uint32_t nxy = static_cast<uint32_t>(a.nx) * a.ny, N = nxy * a.nz;
    const uint32_t fsE = static_cast<uint32_t>(a.fs) * E;
    const uint32_t n0 = static_cast<uint32_t>(b) * NB + threadIdx.x;
    if (static_cast<uint32_t>(b) * NB >= N) return;  // uniform per block
    const bool act = n0 < N;
    const uint32_t n = act ? n0 : N - 1;
    const NodeNbr nb = node_nbr(n, a);
    const uint8_t m = gptr(a.mat)[n] & MAT_ID_MASK;
    const bool fluid = m == MAT_FLUID;
    const bool top = a.evap && nb.z == a.nz - 2;
    S raw[2][Q];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const auto src = make_rsrc(static_cast<const char *>(a.fsrc) + size_t(k) * Q * fsE, Q * fsE);
#pragma unroll
        for (int i = 0; i < Q; ++i) raw[k][i] = buf_load<S>(src, nb.at(-cx(i), -cy(i), -cz(i)) * E, i * fsE);
    }
    C dr[2], j[2][3];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        C fv[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) fv[i] = Codec<S>::dec(raw[k][i]);
        stream_moments(a, k, top, fv, dr[k], j[k]);
    }
    if (act) stream_store<S>(a, n, m, dr, j);
    // the sink's column counts of this step start at zero (the collide pass adds)
    if (a.sink && n0 < nxy) a.h_write[n0] = 0;
    // ledger: this step's streaming moves the stored f*_i(t) with c_iz = +1 of
    // the plane below the reservoir into it and pulls w_i rho_top_k out of it
    book_top(a, b, act && fluid && top, red, [&](int k, int i) {
        const auto src = make_rsrc(static_cast<const char *>(a.fsrc) + size_t(k) * Q * fsE, Q * fsE);
        return Codec<S>::dec(buf_load<S>(src, n * E, i * fsE));
    });
}

// Collides one node per thread of block b.  Returns the mass the sink moved
// from A to B there.
// DST: the new state is kept as moments (a.mom), else as populations (a.fdst).
template <class S, bool SINK = false, bool DST = false>
__device__ __forceinline__ double sc_collide_nodes(const StepArgs &a, int b) {
    using C = typename Codec<S>::C;
    constexpr uint32_t E = sizeof(S);
    const uint32_t nxy = static_cast<uint32_t>(a.nx) * a.ny, N = nxy * a.nz;
    const uint32_t fsE = static_cast<uint32_t>(a.fs) * E;
    const uint32_t n = static_cast<uint32_t>(b) * NB + threadIdx.x;
    if (n >= N) return 0.0;
    const NodeNbr nb = node_nbr(n, a);
    const uint8_t mt = gptr(a.mat)[n];
    const unsigned known = *a.status;  // status bits already raised before this launch
    const C *psi = static_cast<const C *>(a.rho_out);
    const auto pr = [&](int k) { return make_rsrc(psi + size_t(k) * a.fs, uint32_t(a.fs) * uint32_t(sizeof(C))); };
    // sum_i w_i psi(x + c_i) c_i taken over opposite pairs as central
    // differences w_i c_i (psi(x + c_i) - psi(x - c_i)): no cancellation
    C sg[2][3], own[2], above[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const auto r = pr(k);
        C v[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) v[i] = buf_load<C>(r, nb.at(cx(i), cy(i), cz(i)) * uint32_t(sizeof(C)), 0);
        own[k] = v[0];
        above[k] = v[5];
        C sx = C(0), sy = C(0), sz = C(0);
#pragma unroll
        for (int i = 1; i < Q; i += 2) {
            const C d = wgt<C>(i) * (v[i] - v[i + 1]);
            if (cx(i) == 1) sx += d;
            if (cx(i) == -1) sx -= d;
            if (cy(i) == 1) sy += d;
            if (cy(i) == -1) sy -= d;
            if (cz(i) == 1) sz += d;
            if (cz(i) == -1) sz -= d;
        }
        sg[k][0] = sx;
        sg[k][1] = sy;
        sg[k][2] = sz;
    }
    // rod nodes go through the same arithmetic (all their moments are zero,
    // so every deviation they store is exactly zero) and store with the fluid
    // lanes: a wave that a rod cuts through then still writes whole lines,
    // where masked lanes would leave partial lines that HBM has to read,
    // merge and write back.  Nothing reads these slots before the rod passes
    // rewrite them (link) or refill them.
    const uint8_t mid = mt & MAT_ID_MASK;
    if (mid != MAT_FLUID && mid != MAT_ROD) return 0.0;
    const bool fluid = mid == MAT_FLUID;
    const auto dst0 = make_rsrc(a.jm, Q * fsE);
    const C rho[2] = {fluid ? own[0] : C(0), fluid ? own[1] : C(0)};
    C j[3] = {C(0), C(0), C(0)}, dr[2] = {rho[0], rho[1]};
    if (fluid) {
#pragma unroll
        for (int d = 0; d < 3; ++d) j[d] = get_moment<S>(dst0, n * E, fsE, d);
        if (a.rho_ref[0] != 0.0 || a.rho_ref[1] != 0.0) {
            dr[0] = get_moment<S>(dst0, n * E, fsE, 3);
            dr[1] = get_moment<S>(dst0, n * E, fsE, 4);
        }
    }
    // Shan-Chen force: F_k = -G psi_k(x) sum_i w_i psi_kbar(x + c_i) c_i + rho_k g
    C F[2][3];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const C gp = -C(a.G) * rho[k];
#pragma unroll
        for (int d = 0; d < 3; ++d) F[k][d] = gp * sg[1 - k][d] + rho[k] * C(a.g[d]);
    }
    // velocity shift (tau = 1): u' = sum_k j_k / sum_k rho_k; u_k^eq = u' + F_k / rho_k
    const C rt = rho[0] + rho[1];
    const C ir = rt > C(0) ? C(1) / rt : C(0);
    // health check on the physical velocity (sum_k j_k + F/2) / rho
    unsigned st = 0;
    {
        C usq_chk = C(0);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const C ud = (j[d] + C(0.5) * (F[0][d] + F[1][d])) * ir;
            usq_chk += ud * ud;
        }
        if (fluid && !(rt > C(0))) st |= ST_RHO;
        if (fluid && !(usq_chk <= C(0.09))) st |= (usq_chk != usq_chk) ? ST_NAN : ST_SPEED;
    }
    // sink (Eq. 8): a liquid node under a gas fluid node moves min(J, f*_0^A)
    bool sink_if = false;
    C sink_J = C(0), sink_d = C(0);
    if constexpr (SINK) {
        if (fluid && rho[0] > rho[1] && above[0] < above[1] && (a.pz || nb.z + 1 < a.nz) &&
            (gptr(a.mat)[nb.at(0, 0, 1)] & MAT_ID_MASK) == MAT_FLUID) {
            sink_if = true;
            sink_J = C(a.sink_J0) / (C(a.sink_K) + C(gptr(a.h_read)[nb.at(0, 0, 0) - nb.zs[1]]) / C(a.sink_h0));
        }
    }
    const bool near_wall = fluid && (mt & MAT_NEAR_WALL) != 0;
    // 16-bit storage with stochastic rounding: the random bits depend on
    // (node, array, step) only; the wall slots reuse the encoded values
    SrStream sr{0u, 0u};
    if constexpr (sizeof(S) == 2) {
        if (a.sr_key) sr.state = sr_seed(a.sr_key, n);
    }
    auto encode = [&](C v, int arr) -> S {
        if constexpr (sizeof(S) == 2) {
            if (a.sr_key) return Stochastic<S>::enc(v, sr.bits(arr));
        }
        return Codec<S>::enc(v);
    };
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const auto dst = make_rsrc(static_cast<char *>(a.fdst) + size_t(k) * Q * fsE, Q * fsE);
        C ue[3];
        const bool ok = rho[k] >= C(1e-12);
        const C rk = ok ? C(1) / rho[k] : C(0);
#pragma unroll
        for (int d = 0; d < 3; ++d) ue[d] = j[d] * ir + F[k][d] * rk;
        // Eq. 2 with tau = 1: f* = f^eq
        C deq[Q], deq_sum = C(0);
        if constexpr (sizeof(S) == 2) {
            eq_pairs(dr[k], rho[k], ue, deq);
        } else {
            const Eq<C> eq = make_eq(dr[k], rho[k], ue[0], ue[1], ue[2]);
#pragma unroll
            for (int i = 1; i < Q; ++i) deq[i] = eq_pop(i, eq);
        }
#pragma unroll
        for (int i = 1; i < Q; ++i) deq_sum += deq[i];
        deq[0] = dr[k] - deq_sum;
        if constexpr (DST) {
            const C v[4] = {fluid ? dr[k] : pop_mark(C(0)), ue[0], ue[1], ue[2]};
            const auto st = make_rsrc(a.mom, 10 * fsE);
            store_state<S>(st, n, fsE, k, v);
            put_moment<S>(st, n * E, fsE, 8 + k, deq[0]);
            continue;
        }
        S sstar[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            C ds = deq[i];
            if constexpr (SINK) {
                // Eq. 8: min(J, f*_0^A), at least 0, leaves A's rest population for B's
                if (i == 0 && sink_if) {
                    if (k == 0) {
                        sink_d = fmax(fmin(sink_J, ds + wgt<C>(0) * C(a.rho_ref[0])), C(0));
                        ds -= sink_d;
                    } else {
                        ds += sink_d;
                    }
                }
            }
            sstar[i] = encode(ds, k * Q + i);
            buf_store<S>(sstar[i], dst, n * E, i * fsE);
        }
        if (near_wall) {
            // halfway bounce-back: hand f*_j(x) to the wall node x + c_j as
            // direction opp(j) (w_j = w_opp(j), so the deviation carries over)
#pragma unroll
            for (int jd = 1; jd < Q; ++jd) {
                const uint32_t q = nb.at(cx(jd), cy(jd), cz(jd));
                if (is_static_wall(gptr(a.mat)[q] & MAT_ID_MASK)) buf_store<S>(sstar[jd], dst, q * E, opp(jd) * fsE);
            }
        }
    }
    post_status(a.status, known, st);
    if constexpr (SINK) {
        // the column height the next step reads: liquid after the sink (an
        // integer count, so the order of the adds does not matter)
        if (fluid && rho[0] - sink_d > rho[1] + sink_d) atomicAdd(a.h_write + (nb.at(0, 0, 0) - nb.zs[1]), 1);
    }
    return double(sink_d);
}

template <class S>
__global__ void __launch_bounds__(NB) sc_stream_kernel(StepArgs a) {
    sc_stream_nodes<S>(a, xcd_range(blockIdx.x, gridDim.x));
}
// The stream pass from moments.  A work-group takes a brick of XB x YB x ZB
// nodes; the moments of the brick and its ring go to LDS once, as what the
// populations need of a node (A, R and u, see node_access.h), so that the 18 x 2
// evaluations per node read 3 or 4 values each.  The work-groups past the
// bricks book the streaming's exchange with the reservoir.
//
// Against the pass over populations it reads 40 bytes per FP32 node instead of
// 152, and the collision behind it stores 40 instead of 152; what bounds it is
// the evaluation (about 450 vector and 140 LDS instructions per node).  Per step
// in a call of many, populations -> moments:
//   FP32 256 x 128 x 64: 124 -> 66 us (48 + 27 in the profiler's clocks);
//     128 x 64 x 64: 33 -> 26; 117 x 51 x 37: 18.3 -> 17.4
//   FP64 256 x 128 x 64: 304 -> 138 us; 128 x 64 x 64: 64 -> 43; 32^3: 14.5 -> 13
// (128 x 64 x 32 alone is even in FP32, 18.8 -> 19.5).  Which calls of two steps or
// more take it, and why the line lies there: moment_chain in lbm_api.hip.  Bricks of 32 x 4 x 4 are as fast on large lattices and
// 8 percent slower on the ragged one; reading the neighbours' moments through L1
// instead of LDS: 61 us for the pass, before the rest population had its array.
constexpr int XB = 32, YB = 4, ZB = 2, BT = XB * YB * ZB;
constexpr int XH = XB + 2, YH = YB + 2, ZH = ZB + 2, BH = XH * YH * ZH;
static_assert(BT == NB, "the booking work-groups take blocks of NB nodes");
__host__ __device__ int state_bricks(int nx, int ny, int nz) {
    return ((nx + XB - 1) / XB) * ((ny + YB - 1) / YB) * ((nz + ZB - 1) / ZB);
}

template <class S>
__device__ __forceinline__ void sc_stream_state(const StepArgs &a, int b) {
    using C = S;  // FP32 and FP64 storage only
    constexpr uint32_t E = sizeof(S);
    extern __shared__ char lds_raw[];
    __shared__ int wmark[BT / 64];
    __shared__ double led[NB / 64][2];
    C *sh = reinterpret_cast<C *>(lds_raw);  // [2][A, R, ux, uy, uz][BH]
    auto val = [&](int k, int q, int h) -> C & { return sh[(5 * k + q) * BH + h]; };
    const int nbx = (a.nx + XB - 1) / XB, nby = (a.ny + YB - 1) / YB, nbr = state_bricks(a.nx, a.ny, a.nz);
    const uint32_t nxy = static_cast<uint32_t>(a.nx) * a.ny, fsE = static_cast<uint32_t>(a.fs) * E;
    const C rref[2] = {C(a.rho_ref[0]), C(a.rho_ref[1])};
    const auto st = make_rsrc(a.mom, 10 * fsE);
    const auto src = [&](int k) { return make_rsrc(static_cast<const char *>(a.fsrc) + size_t(k) * Q * fsE, Q * fsE); };
    if (b >= nbr) {  // uniform per block
        const int bb = b - nbr + int(uint32_t(a.nz - 2) * nxy / NB);
        const uint32_t n = static_cast<uint32_t>(bb) * NB + threadIdx.x;
        const bool here = n / nxy + 2 == static_cast<uint32_t>(a.nz) &&
                          (gptr(a.mat)[n] & MAT_ID_MASK) == MAT_FLUID;
        book_top(a, bb, here, led, [&](int k, int i) {
            C v[4], v0[4];
            load_state<S>(st, n, fsE, k, v);
            load_state<S>(st, n, fsE, 0, v0);
            const C f = buf_load<S>(src(k), n * E, i * fsE);
            return is_pop_mark(v0[0]) ? f : eq_pop(i, make_eq(v[0], rref[k] + v[0], v[1], v[2], v[3]));
        });
        return;
    }
    // z fastest: an XCD's range is whole columns, so that rods lying on the
    // substrate are shared out (in z slabs they would be one XCD's)
    const int nbz = nbr / (nbx * nby), col = b / nbz;
    const int x0 = col % nbx * XB, y0 = col / nbx * YB, z0 = (b - col * nbz) * ZB;
    // coordinate of the ring: wrapped, or clamped where nothing reads it
    auto at = [](int v, int n, int per) {
        const int lo = per ? n - 1 : 0, hi = per ? 0 : n - 1;
        return v < 0 ? lo : (v >= n ? hi : v);
    };
    // the brick and its ring by rows of XH nodes: XB of a row by XB threads, then
    // the rows' two ends by the first threads
    static_assert(YH * ZH % (BT / XB) == 0 && 2 * YH * ZH <= BT, "rows dealt evenly, their ends in one go");
    constexpr int RL = YH * ZH / (BT / XB);
    const int tx = threadIdx.x % XB, tr = threadIdx.x / XB;
    const auto row = [&](int r) {
        return uint32_t(at(min(z0 - 1 + r / YH, a.nz), a.nz, a.pz)) * nxy +
               uint32_t(at(min(y0 - 1 + r % YH, a.ny), a.ny, a.py)) * a.nx;
    };
    const uint32_t xm = at(min(x0 + tx, a.nx), a.nx, a.px);
    const bool ends = threadIdx.x < 2 * YH * ZH;
    const int er = threadIdx.x >> 1, eh = er * XH + (threadIdx.x & 1 ? XB + 1 : 0);
    C v[RL][2][4], ve[2][4];
#pragma unroll
    for (int l = 0; l < RL; ++l) {
        const uint32_t q = row(tr + l * (BT / XB)) + xm;
#pragma unroll
        for (int k = 0; k < 2; ++k) load_state<S>(st, q, fsE, k, v[l][k]);
    }
    if (ends) {
        const uint32_t q = row(er) + at(min(x0 + (threadIdx.x & 1 ? XB : -1), a.nx), a.nx, a.px);
#pragma unroll
        for (int k = 0; k < 2; ++k) load_state<S>(st, q, fsE, k, ve[k]);
    }
    const int ty = tr % YB, tz = tr / YB;
    const int x = x0 + tx, y = y0 + ty, z = z0 + tz;
    const bool act = x < a.nx && y < a.ny && z < a.nz;
    const uint32_t n = act ? uint32_t(z) * nxy + uint32_t(y) * a.nx + x : 0;
    const uint8_t mt = gptr(a.mat)[n], m = mt & MAT_ID_MASK;
    const C rest[2] = {get_moment<S>(st, n * E, fsE, 8), get_moment<S>(st, n * E, fsE, 9)};
    bool mark = false;
    const auto put = [&](int h, const C(&w2)[2][4]) {
        const bool mk = is_pop_mark(w2[0][0]);
        mark |= mk;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const C *w = w2[k];
            const Eq<C> e = make_eq(w[0], rref[k] + w[0], w[1], w[2], w[3]);
            val(k, 0, h) = k == 0 && mk ? w[0] : e.A;
            val(k, 1, h) = e.R;
#pragma unroll
            for (int d = 0; d < 3; ++d) val(k, 2 + d, h) = e.u[d];
        }
    };
#pragma unroll
    for (int l = 0; l < RL; ++l) put((tr + l * (BT / XB)) * XH + 1 + tx, v[l]);
    if (ends) put(eh, ve);
    const bool any = __any(mark);
    if ((threadIdx.x & 63) == 0) wmark[threadIdx.x >> 6] = any;
    __syncthreads();
    bool marks = false;  // the brick or its ring holds a marked node
#pragma unroll
    for (int q = 0; q < BT / 64; ++q) marks |= wmark[q] != 0;
    if (!act) return;
    const int hc = ((tz + 1) * YH + ty + 1) * XH + tx + 1;
    const bool fluid = m == MAT_FLUID, top = a.evap && z == a.nz - 2;
    const auto ring = [&](int i) { return hc - ((cz(i) * YH + cy(i)) * XH + cx(i)); };
    const NodeNbr nb = node_nbr(x, y, z, a);
    const auto nbr_at = [&](int i) { return nb.at(-cx(i), -cy(i), -cz(i)); };
    // directions that come from a static wall, and from a marked node (bit 0: this one)
    unsigned walls = 0, slots = 0;
    if (fluid && (mt & MAT_NEAR_WALL)) {
        uint8_t mq[Q];
#pragma unroll
        for (int i = 1; i < Q; ++i) mq[i] = gptr(a.mat)[nbr_at(i)] & MAT_ID_MASK;
#pragma unroll
        for (int i = 1; i < Q; ++i) walls |= is_static_wall(mq[i]) ? 1u << i : 0u;
    }
    if (marks && fluid) {
#pragma unroll
        for (int i = 0; i < Q; ++i) slots |= is_pop_mark(val(0, 0, ring(i))) ? 1u << i : 0u;
    }
    C dr[2], j[2][3];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        C fv[Q];
        fv[0] = rest[k];
#pragma unroll
        for (int i = 1; i < Q; ++i) {
            const int h = ring(i);
            fv[i] = eq_pop_full(i, val(k, 0, h), val(k, 1, h), [&](int d) { return val(k, 2 + d, h); });
        }
        // halfway bounce-back: from a static wall comes the node's own f*_opp(i)
        if (walls) {
            const Eq<C> e{val(k, 0, hc), val(k, 1, hc), {val(k, 2, hc), val(k, 3, hc), val(k, 4, hc)}};
#pragma unroll
            for (int i = 1; i < Q; ++i) fv[i] = (walls >> i) & 1u ? eq_pop_full(opp(i), e) : fv[i];
        }
        // from a marked node the element of its population; directions without one
        // read the node's first element again, so that all loads are in flight
        // together and cost no lines of their own
        if (slots) {
            // a marked node's own populations are what its walls return
            const unsigned far = slots & ~walls, self = slots & 1u ? walls : 0u;
            S slot[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                uint32_t v = n * E;
                v = far >> i & 1u ? nbr_at(i) * E + i * fsE : v;
                v = self >> i & 1u ? n * E + opp(i) * fsE : v;
                slot[i] = buf_load<S>(src(k), v, 0);
            }
#pragma unroll
            for (int i = 0; i < Q; ++i)
                fv[i] = (far | self) >> i & 1u ? (i > 6 ? C(2) : C(1)) * Codec<S>::dec(slot[i]) : fv[i];
        }
        stream_moments<true>(a, k, top, fv, dr[k], j[k]);
    }
    stream_store<S>(a, n, m, dr, j);
}

template <class S>
__global__ void __launch_bounds__(BT, sizeof(S) == 4 ? 5 : 2) sc_stream_state_kernel(StepArgs a) {
    // the booking work-groups first (they are a few long chains), then the bricks
    // in XCD order
    const int nbr = state_bricks(a.nx, a.ny, a.nz), n8 = (nbr + 7) & ~7, nbk = gridDim.x - n8, g = blockIdx.x;
    const int b = g < nbk ? nbr + g : xcd_range(g - nbk, n8);
    if (g >= nbk && b >= nbr) return;
    sc_stream_state<S>(a, b);
}
template <class S, bool SINK, bool DST>
__global__ void __launch_bounds__(NB) sc_collide_kernel(StepArgs a) {
    const int b = xcd_range(blockIdx.x, gridDim.x);
    const double mv = sc_collide_nodes<S, SINK, DST>(a, b);
    if constexpr (SINK) {
        // the block's moved mass into its own ledger pair (A loses it, B gains it)
        __shared__ double red[NB / 64];
        const double w = wave_sum(mv);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = w;
        __syncthreads();
        if (threadIdx.x == 0 && b < split_blocks(a.nx, a.ny, a.nz)) {
            double sum = 0.0;
            for (int q = 0; q < NB / 64; ++q) sum += red[q];
            a.sink_ledger[2 * size_t(b)] += sum;
            a.sink_ledger[2 * size_t(b) + 1] -= sum;
        }
    }
}
// batches: a work list of (lattice, block of NB nodes) entries
template <class S>
__global__ void __launch_bounds__(NB) sc_stream_batch_kernel(const StepArgs *__restrict__ all,
                                                             const int2 *__restrict__ work) {
    const int2 w = work[blockIdx.x];
    if (w.x < 0) return;  // padding entry, uniform per block
    const StepArgs a = all[w.x];
    sc_stream_nodes<S>(a, w.y);
}
template <class S, bool DST>
__global__ void __launch_bounds__(NB) sc_collide_batch_kernel(const StepArgs *__restrict__ all,
                                                              const int2 *__restrict__ work) {
    const int2 w = work[blockIdx.x];
    if (w.x < 0) return;
    const StepArgs a = all[w.x];
    sc_collide_nodes<S, false, DST>(a, w.y);
}
// the stream pass from moments: entries (lattice, brick), and past the bricks
// (lattice, bricks + booking block)
template <class S>
__global__ void __launch_bounds__(BT, sizeof(S) == 4 ? 5 : 2)
    sc_stream_state_batch_kernel(const StepArgs *__restrict__ all, const int2 *__restrict__ work) {
    const int2 w = work[blockIdx.x];
    if (w.x < 0) return;
    const StepArgs a = all[w.x];
    sc_stream_state<S>(a, w.y);
}

// work-groups that book the plane below the reservoir: blocks of NB nodes
int book_blocks(int nx, int ny, int nz, int evap) {
    const int64_t nxy = int64_t(nx) * ny;
    return evap ? int(((nz - 1) * nxy - 1) / NB - (nz - 2) * nxy / NB) + 1 : 0;
}
template <class S>
static hipError_t launch_split(const StepArgs &a, bool src, bool dst, hipStream_t s) {
    const dim3 grid((split_blocks(a.nx, a.ny, a.nz) + 7) & ~7), block(NB);
    if ((a.sink || src || dst) && sizeof(S) < 4) return hipErrorInvalidValue;
    if (a.sink && (src || dst)) return hipErrorInvalidValue;
    auto collide = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, block, 0, s, a);
        return hipGetLastError();
    };
    if constexpr (sizeof(S) >= 4) {
        if (src) {
            const int nbr = (state_bricks(a.nx, a.ny, a.nz) + 7) & ~7;
            hipLaunchKernelGGL((sc_stream_state_kernel<S>), dim3(nbr + book_blocks(a.nx, a.ny, a.nz, a.evap)), dim3(BT),
                               10 * BH * sizeof(S), s, a);
        }
    }
    if (!src) hipLaunchKernelGGL((sc_stream_kernel<S>), grid, block, 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if constexpr (sizeof(S) >= 4) {  // the sink and the state as moments: FP32 or FP64 storage
        if (a.sink) return collide(sc_collide_kernel<S, true, false>);
        if (dst) return collide(sc_collide_kernel<S, false, true>);
    }
    return collide(sc_collide_kernel<S, false, false>);
}
template <class S>
static hipError_t launch_split_batch(const StepArgs *all, const int2 *work, int nwork, const int2 *swork, int nswork,
                                     bool src, bool dst, hipStream_t s) {
    if ((src || dst) && sizeof(S) < 4) return hipErrorInvalidValue;
    if constexpr (sizeof(S) >= 4) {
        if (src)
            hipLaunchKernelGGL((sc_stream_state_batch_kernel<S>), dim3(nswork), dim3(BT), 10 * BH * sizeof(S), s, all,
                               swork);
    }
    if (!src) hipLaunchKernelGGL((sc_stream_batch_kernel<S>), dim3(nwork), dim3(NB), 0, s, all, work);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if constexpr (sizeof(S) >= 4) {
        if (dst) {
            hipLaunchKernelGGL((sc_collide_batch_kernel<S, true>), dim3(nwork), dim3(NB), 0, s, all, work);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((sc_collide_batch_kernel<S, false>), dim3(nwork), dim3(NB), 0, s, all, work);
    return hipGetLastError();
}

hipError_t launch_sc_split(int prec, const StepArgs &a, bool src, bool dst, hipStream_t s) {
    switch (prec) {
        case LB_F64:
            return launch_split<double>(a, src, dst, s);
        case LB_F32:
            return launch_split<float>(a, src, dst, s);
        case LB_F16DEV:
            return launch_split<_Float16>(a, src, dst, s);
        case LB_BF16DEV:
            return launch_split<bf16_t>(a, src, dst, s);
        default:
            return hipErrorInvalidValue;
    }
}
hipError_t launch_sc_split_batch(int prec, const StepArgs *all, const int2 *work, int nwork,
                                 const int2 *swork, int nswork, bool src, bool dst, hipStream_t s) {
    switch (prec) {
        case LB_F64:
            return launch_split_batch<double>(all, work, nwork, swork, nswork, src, dst, s);
        case LB_F32:
            return launch_split_batch<float>(all, work, nwork, swork, nswork, src, dst, s);
        case LB_F16DEV:
            return launch_split_batch<_Float16>(all, work, nwork, swork, nswork, src, dst, s);
        case LB_BF16DEV:
            return launch_split_batch<bf16_t>(all, work, nwork, swork, nswork, src, dst, s);
        default:
            return hipErrorInvalidValue;
    }
}

int tiles_xy(int nx, int ny, int tile_y) { return ((nx + 63) / 64) * ((ny + tile_y - 1) / tile_y); }

template <class S, int TY, bool SINK>
static hipError_t launch_one(const StepArgs &a, hipStream_t s) {
    const int nblk = a.ntx * a.nty * a.nzc;
    hipLaunchKernelGGL((sc_step_kernel<S, TY, SINK>), dim3(nblk), dim3(64 * TY), 0, s, a);
    return hipGetLastError();
}

// The fused step runs where the two-pass step does not, with tau != 1: the
// tiles of one row per thread, whose registers hold the populations.
template <class S>
static hipError_t launch_prec(const TileCfg &t, const StepArgs &a, hipStream_t s) {
    const int ty = t.tile_y, rp = t.rows_per_thread;
    if (rp != 1) return hipErrorInvalidValue;
    if (a.sink) {
        if constexpr (std::is_same_v<S, float>) {  // FP64 runs the sink with tau = 1 only
            if (ty == 4) return launch_one<S, 4, true>(a, s);
            if (ty == 8) return launch_one<S, 8, true>(a, s);
        }
        return hipErrorInvalidValue;
    }
    if (ty == 4) return launch_one<S, 4, false>(a, s);
    if (ty == 8) return launch_one<S, 8, false>(a, s);
    return hipErrorInvalidValue;
}

template <class S>
static hipError_t launch_batch_prec(const TileCfg &t, const StepArgs *all, const int2 *work, int nwork, hipStream_t s) {
    if (t.rows_per_thread != 1) return hipErrorInvalidValue;
    if (t.tile_y == 4) {
        hipLaunchKernelGGL((sc_step_batch_kernel<S, 4>), dim3(nwork), dim3(64 * 4), 0, s, all, work);
    } else if (t.tile_y == 8) {
        hipLaunchKernelGGL((sc_step_batch_kernel<S, 8>), dim3(nwork), dim3(64 * 8), 0, s, all, work);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_sc_step_batch(int prec, const TileCfg &t, const StepArgs *all, const int2 *work, int nwork,
                                hipStream_t s) {
    switch (prec) {
        case LB_F64:
            return launch_batch_prec<double>(t, all, work, nwork, s);
        case LB_F32:
            return launch_batch_prec<float>(t, all, work, nwork, s);
        case LB_F16DEV:
            return launch_batch_prec<_Float16>(t, all, work, nwork, s);
        case LB_BF16DEV:
            return launch_batch_prec<bf16_t>(t, all, work, nwork, s);
        default:
            return hipErrorInvalidValue;
    }
}

hipError_t launch_sc_step(int prec, const TileCfg &t, const StepArgs &a, hipStream_t s) {
    switch (prec) {
        case LB_F64:
            return launch_prec<double>(t, a, s);
        case LB_F32:
            return launch_prec<float>(t, a, s);
        case LB_F16DEV:
            return launch_prec<_Float16>(t, a, s);
        case LB_BF16DEV:
            return launch_prec<bf16_t>(t, a, s);
        default:
            return hipErrorInvalidValue;
    }
}

}  // namespace lbm
