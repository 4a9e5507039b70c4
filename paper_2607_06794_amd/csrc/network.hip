// Resistor network of a deposit (Methods, electrical characterisation,
// Eqs. 15-18): beads joined below a cutoff distance with conductance 1/r,
// potentials from Kirchhoff's current law between two electrodes along x,
// node currents and the current leaving the source.
//
// The network is small next to the lattice (a few thousand beads per
// deposit), so the solve is latency-bound, not bandwidth-bound:
//  * neighbours: one wavefront per bead scans every bead in index order (a
//    deterministic, ascending neighbour list per bead);
//  * Kirchhoff: a Jacobi-preconditioned conjugate-gradient solve in one
//    work-group; each iteration costs one sparse product and two work-group
//    reductions in a fixed order, and the loop is bounded by the caller's
//    iteration limit.  Up to NET_ROWS beads the rows are sorted by length and
//    their vectors kept in registers; beyond, the vectors live in L2 and the
//    search direction in LDS (up to NET_LDS_P beads).
#include <hip/hip_runtime.h>

#include <mutex>

#include "lbm.h"
#include "lbm_device.h"
#include "lbm_internal.h"

namespace lbm {

// Fixed scratch of lb_kirchhoff_noalloc: the workspace of a network of up to
// LB_NET_NOALLOC_MAX_BEADS beads, one copy per GPU for the life of the
// process.  Host code never uses this name as an address (on the host it is a
// stand-in symbol); net_static_scratch() returns the device address.
static __device__ __align__(256) char net_scratch[net_workspace_bytes(LB_NET_NOALLOC_MAX_BEADS)];

hipError_t net_static_scratch(void **ptr, size_t *bytes) {
    constexpr int MAX_DEV = 64;
    static std::mutex mu;
    static void *addr[MAX_DEV] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEV) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(net_scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    *bytes = sizeof(net_scratch);
    return hipSuccess;
}

void net_carve(NetArgs &a, void *ws) {
    const size_t nn = size_t(a.n);
    char *w = static_cast<char *>(ws);
    // doubles first (8-byte aligned from the 256-byte aligned base), then the ints
    a.g = reinterpret_cast<double *>(w);
    w += nn * NET_DEG * sizeof(double);
    a.diag = reinterpret_cast<double *>(w);
    a.r = a.diag + nn;
    a.z = a.r + nn;
    a.p = a.z + nn;
    a.q = a.p + nn;
    a.out = a.q + nn;
    w += 5 * nn * sizeof(double) + 8 * sizeof(double);
    a.nbr = reinterpret_cast<int *>(w);
    a.deg = a.nbr + nn * NET_DEG;
    a.cls = a.deg + nn;
    a.cnt = a.cls + nn;
}

namespace {

constexpr int NET_TB = 256;   // threads per work-group of the neighbour scan
constexpr int NET_CG = 1024;  // threads of the solve's single work-group

__device__ inline int net_class(double x, const NetArgs &a) { return x < a.x_src ? 1 : (x > a.x_snk ? 2 : 0); }

// every thread gets the work-group sum of v[q]: xor butterfly per
// wavefront, then the wavefront sums added in order
template <int NV>
__device__ inline void wg_sum(double (&v)[NV], double *sh) {
#pragma unroll
    for (int q = 0; q < NV; ++q)
#pragma unroll
        for (int s = 32; s > 0; s >>= 1) v[q] += __shfl_xor(v[q], s, 64);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    __syncthreads();  // earlier readers of sh are done
    if (l == 0)
#pragma unroll
        for (int q = 0; q < NV; ++q) sh[q * (NET_CG / 64) + w] = v[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        double t = 0.0;
        for (int k = 0; k < NET_CG / 64; ++k) t += sh[q * (NET_CG / 64) + k];
        v[q] = t;
    }
}

// r_ij^2 = (dx^2 + dy^2) + dz^2 without contraction: the edge decision is
// taken exactly as stated
__device__ inline double net_r2(const double *pi, const double *pj) {
    const double dx = pj[0] - pi[0], dy = pj[1] - pi[1], dz = pj[2] - pi[2];
    return __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
}

// Beads j != i with 0 < r_ij^2 < r_c^2, ascending j; deg may exceed NET_DEG
// (only the first NET_DEG are stored; the host reports the excess).  One
// wavefront for PB beads, 64 candidates at a time, compacted by ballots: with one
// thread per bead the scan was a chain of n tests on n / 256 work-groups
// (314 us for 3 300 beads; now 18).  PB = 1 while that leaves CUs idle; beyond
// NET_ROWS each candidate's loads serve four beads (65 536 beads, the call with one
// iteration: 10.6 -> 5.4 ms; the scan by threads 8.2).
// ROWS: the lists of the row-sorted solve, as 16-bit indices (the conductances
// follow when the rows are laid out).
template <bool ROWS, int PB>
__global__ void __launch_bounds__(NET_TB) net_edges_kernel(NetArgs a) {
    const int i0 = (blockIdx.x * (NET_TB / 64) + int(threadIdx.x >> 6)) * PB, lane = threadIdx.x & 63;
    if (i0 >= a.n) return;  // uniform per wavefront
    double own[PB][3];
    int k[PB];
#pragma unroll
    for (int b = 0; b < PB; ++b) {
        k[b] = 0;
        for (int d = 0; d < 3; ++d) own[b][d] = a.pos[3 * min(i0 + b, a.n - 1) + d];
    }
    for (int j0 = 0; j0 < a.n; j0 += 64) {
        const int j = min(j0 + lane, a.n - 1);
        const double pj[3] = {a.pos[3 * j], a.pos[3 * j + 1], a.pos[3 * j + 2]};
#pragma unroll
        for (int b = 0; b < PB; ++b) {
            const int i = i0 + b;
            const double r2 = net_r2(own[b], pj);
            const bool hit = i < a.n && j0 + lane < a.n && r2 > 0.0 && r2 < a.rc2;
            const uint64_t m = __ballot(hit);
            const int at = k[b] + __popcll(m & ((uint64_t(1) << lane) - 1));
            if (hit && at < NET_DEG) {
                if constexpr (ROWS) {
                    reinterpret_cast<uint16_t *>(a.nbr)[size_t(i) * NET_DEG + at] = uint16_t(j);
                } else {
                    a.nbr[size_t(i) * NET_DEG + at] = j;
                    a.g[size_t(i) * NET_DEG + at] = 1.0 / sqrt(r2);
                }
            }
            k[b] += __popcll(m);
        }
    }
#pragma unroll
    for (int b = 0; b < PB; ++b)
        if (lane == 0 && i0 + b < a.n) a.deg[i0 + b] = k[b];
}

// ---------------------------------------------------------------------------
// Networks of up to NET_ROWS beads: the rows sorted by degree (ties in bead
// order), so that the 64 rows of a wavefront have nearly equal lengths, and
// laid out edge-major: conductance k of the row of rank q at g[k n + q], eight
// times its neighbour's bead index (the byte offset of a vector element) the
// 16-bit half k & 1 of cols[(k / 2) n + q].  A wavefront then reads 64 rows'
// next edges from consecutive addresses.  Past its end a row is filled with
// edges of no conductance to bead 0, so the product needs no bounds.
// ---------------------------------------------------------------------------
constexpr int NET_ROWS = 8192;

__device__ inline uint32_t *net_cols(const NetArgs &a) {
    // the second half of the neighbour array; the 16-bit lists are its first
    return reinterpret_cast<uint32_t *>(a.nbr) + size_t(a.n) * (NET_DEG / 2);
}

// one wavefront per bead: its rank, then its row
__global__ void __launch_bounds__(NET_TB) net_rows_kernel(NetArgs a) {
    const int i = blockIdx.x * (NET_TB / 64) + int(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (i >= a.n) return;  // uniform per wavefront
    const int di = min(a.deg[i], NET_DEG);
    int before = 0;
    for (int j0 = 0; j0 < a.n; j0 += 64) {
        const int j = j0 + lane, dj = j < a.n ? min(a.deg[j], NET_DEG) : -1;
        before += __popcll(__ballot(dj > di || (dj == di && j < i)));
    }
    if (lane == 0) a.cls[before] = i;  // the bead of each rank
    const int j = lane < di ? reinterpret_cast<const uint16_t *>(a.nbr)[size_t(i) * NET_DEG + lane] : 0;
    a.g[size_t(lane) * a.n + before] = lane < di ? 1.0 / sqrt(net_r2(a.pos + 3 * i, a.pos + 3 * j)) : 0.0;
    reinterpret_cast<uint16_t *>(net_cols(a))[(size_t(lane >> 1) * a.n + before) * 2 + (lane & 1)] = uint16_t(8 * j);
}

// v plus its neighbour N lanes on within each row of 16 (rotated); over N = 8,
// 4, 2, 1 every lane gets the same sum of its row
template <int N>
__device__ inline double row_add(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 + N, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 + N, 0xF, 0xF, true);
    return v + __hiloint2double(hi, lo);
}
__device__ inline double row_sum(double v) { return row_add<1>(row_add<2>(row_add<4>(row_add<8>(v)))); }
__device__ inline double lane_value(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Work-group sums of v[q] over 16 wavefronts in a fixed order, the same in
// every thread.  One barrier: sh (64 doubles per value) must not be the array
// of the previous sum, whose readers may still be at it.
template <int NV>
__device__ inline void group_sum(double (&v)[NV], double *sh) {
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        v[q] = row_sum(v[q]);
        if ((l & 15) == 0) sh[q * 64 + w * 4 + (l >> 4)] = v[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        const double t = row_sum(sh[q * 64 + l]);
        v[q] = (lane_value(t, 0) + lane_value(t, 16)) + (lane_value(t, 32) + lane_value(t, 48));
    }
}

// Potentials, node currents and the current leaving the source, as
// net_solve_kernel below, in one work-group whose thread t owns the rows of
// rank t, t + 1024, ...: their vectors stay in registers (the potentials and
// the search direction, which every neighbour reads, in LDS) and the matrix
// streams from L2 coalesced.  Bound by one CU's throughput on that stream and
// on the LDS gather: per wavefront and edge about 10 + 12 cycles, 0.55 MB and
// 860 gathers per iteration for 3 300 beads with 55 000 directed edges.  There
// a call takes 2.8 ms (9.8 us per iteration) against 7.5 ms with the vectors
// in L2 and rows of unequal length side by side; 8 140 beads 11.6 against
// 27.4 ms.
template <int R>
__global__ void __launch_bounds__(NET_CG) net_rows_solve_kernel(NetArgs a) {
    __shared__ double sh[3][128];
    extern __shared__ double P[];
    const int n = a.n, t = threadIdx.x;
    double *X = P + n;  // the potentials by rank, each touched by its owner only
    const uint32_t *cols = net_cols(a);
    if (t < 4) a.cnt[t] = 0;
    int row[R], bead[R], dk[R];
    bool fr[R];
    double r[R], p[R], dg[R], q[R];
    double s0[2] = {0.0, 0.0};  // r.z, r.r
    int maxdeg = 0, nsrc = 0, nsnk = 0, dsum = 0;
    __syncthreads();
#pragma unroll
    for (int s = 0; s < R; ++s) {
        const int rk = t + s * NET_CG;
        const bool have = rk < n;
        row[s] = min(rk, n - 1);
        bead[s] = a.cls[row[s]];
        const int d = have ? a.deg[bead[s]] : 0;
        dk[s] = min(d, NET_DEG);
        const int ci = net_class(a.pos[3 * bead[s]], a);
        fr[s] = have && ci == 0;
        double b = 0.0;
        dg[s] = 0.0;
        for (int k = 0; k < dk[s]; ++k) {
            const uint32_t c = cols[size_t(k >> 1) * n + row[s]];
            const int j = (k & 1 ? int(c >> 16) : int(c & 0xFFFFu)) >> 3;
            const double gk = a.g[size_t(k) * n + row[s]];
            dg[s] += gk;
            if (net_class(a.pos[3 * j], a) == 1) b += gk * a.dV;
        }
        if (have) X[row[s]] = ci == 1 ? a.dV : 0.0;
        r[s] = fr[s] ? b : 0.0;
        p[s] = fr[s] && dg[s] > 0.0 ? r[s] / dg[s] : 0.0;
        if (have) P[bead[s]] = p[s];
        s0[0] += r[s] * p[s];
        s0[1] += r[s] * r[s];
        maxdeg = max(maxdeg, d);
        nsrc += have && ci == 1;
        nsnk += have && ci == 2;
        dsum += dk[s];  // the stored edges (a degree above NET_DEG is rejected)
    }
    atomicMax(&a.cnt[0], maxdeg);
    atomicAdd(&a.cnt[1], nsrc);
    atomicAdd(&a.cnt[2], nsnk);
    atomicAdd(&a.cnt[3], dsum);
    group_sum(s0, sh[0]);  // its barrier also publishes P
    double rz = s0[0], rr = s0[1];
    const double bb = s0[1], stop2 = a.tol * a.tol * bb;
    int it = 0;
    while (it < a.max_iter && rr > stop2) {
        double pq[1] = {0.0};
#pragma unroll
        for (int s = 0; s < R; ++s) {
            double off = 0.0;
            const int width = __builtin_amdgcn_readfirstlane(dk[s]);  // the first lane's row is the longest
            for (int k = 0; k < width; k += 4) {  // (eight at a time: 3.05 ms, the rows' ends cost more)
                uint32_t c[2];
                double g[4];
#pragma unroll
                for (int e = 0; e < 2; ++e) c[e] = cols[size_t((k >> 1) + e) * n + row[s]];
#pragma unroll
                for (int e = 0; e < 4; ++e) g[e] = a.g[size_t(k + e) * n + row[s]];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t at = e & 1 ? c[e >> 1] >> 16 : c[e >> 1] & 0xFFFFu;
                    off += g[e] * *reinterpret_cast<const double *>(reinterpret_cast<const char *>(P) + at);
                }
            }
            q[s] = fr[s] ? dg[s] * p[s] - off : 0.0;
            pq[0] += p[s] * q[s];
        }
        group_sum(pq, sh[1]);
        if (!(pq[0] > 0.0)) break;  // same value in every thread
        const double alpha = rz / pq[0];
        double s1[2] = {0.0, 0.0};
#pragma unroll
        for (int s = 0; s < R; ++s) {
            if (!fr[s]) continue;
            r[s] -= alpha * q[s];
            X[row[s]] += alpha * p[s];
            q[s] = dg[s] > 0.0 ? r[s] / dg[s] : 0.0;  // z
            s1[0] += r[s] * q[s];
            s1[1] += r[s] * r[s];
        }
        group_sum(s1, sh[2]);
        const double beta = rz > 0.0 ? s1[0] / rz : 0.0;
        rz = s1[0];
        rr = s1[1];
#pragma unroll
        for (int s = 0; s < R; ++s)
            if (fr[s]) {
                p[s] = q[s] + beta * p[s];
                P[bead[s]] = p[s];
            }
        __syncthreads();  // the next product reads every bead's p
        ++it;
    }
    __syncthreads();
    // Eq. 15 and the current leaving the source electrode
#pragma unroll
    for (int s = 0; s < R; ++s)
        if (t + s * NET_CG < n) {
            P[bead[s]] = X[row[s]];
            a.V[bead[s]] = X[row[s]];
        }
    __syncthreads();
    double st[1] = {0.0};
#pragma unroll
    for (int s = 0; s < R; ++s) {
        const bool src = t + s * NET_CG < n && net_class(a.pos[3 * bead[s]], a) == 1;
        const double xs = X[row[s]];
        double sum = 0.0;
        for (int k = 0; k < dk[s]; ++k) {
            const uint32_t c = cols[size_t(k >> 1) * n + row[s]];
            const int j = (k & 1 ? int(c >> 16) : int(c & 0xFFFFu)) >> 3;
            const double e = a.g[size_t(k) * n + row[s]] * (xs - P[j]);
            sum += fabs(e);
            if (src && net_class(a.pos[3 * j], a) != 1) st[0] += e;
        }
        if (t + s * NET_CG < n) a.I[bead[s]] = 0.5 * sum;
    }
    group_sum(st, sh[0]);
    if (t == 0) {
        a.out[0] = st[0];
        a.out[1] = bb > 0.0 ? sqrt(rr / bb) : 0.0;
        a.out[2] = double(it);
    }
}

// Networks of up to NET_LDS_P beads keep the search direction p in LDS for
// the whole solve: the sparse product reads p at every neighbour, and from
// LDS that read no longer waits on the load of the neighbour's index from L2.
constexpr int NET_LDS_P = 16384;

// potentials (Jacobi-preconditioned CG on the free beads; the electrode beads
// are fixed), then Eq. 15's node currents and the current leaving the source
template <bool LP>
__global__ void __launch_bounds__(NET_CG) net_solve_kernel(NetArgs a) {
    __shared__ double sh[4 * (NET_CG / 64)];
    extern __shared__ double lds_p[];
    double *P = LP ? lds_p : a.p;
    const int n = a.n;
    if (threadIdx.x == 0) {
        for (int q = 0; q < 4; ++q) a.cnt[q] = 0;
    }
    __syncthreads();
    // set-up: x0 = 0 on the free beads, r0 = b = sum over source neighbours of G dV
    double s0[2] = {0.0, 0.0};  // r.z, r.r
    int maxdeg = 0, nsrc = 0, nsnk = 0, dsum = 0;
    for (int i = threadIdx.x; i < n; i += NET_CG) {
        const int ci = net_class(a.pos[3 * i], a);
        const int d = a.deg[i], dk = min(d, NET_DEG);
        double dg = 0.0, b = 0.0;
        for (int k = 0; k < dk; ++k) {
            const int j = a.nbr[size_t(i) * NET_DEG + k];
            const double gk = a.g[size_t(i) * NET_DEG + k];
            dg += gk;
            if (net_class(a.pos[3 * j], a) == 1) b += gk * a.dV;
        }
        a.cls[i] = ci;
        const bool fr = ci == 0;
        const double r = fr ? b : 0.0;
        const double z = (fr && dg > 0.0) ? r / dg : 0.0;
        a.diag[i] = dg;
        a.V[i] = ci == 1 ? a.dV : 0.0;
        a.r[i] = r;
        a.z[i] = z;
        P[i] = z;
        s0[0] += r * z;
        s0[1] += r * r;
        maxdeg = max(maxdeg, d);
        nsrc += ci == 1;
        nsnk += ci == 2;
        dsum += dk;  // the stored edges (a degree above NET_DEG is rejected)
    }
    atomicMax(&a.cnt[0], maxdeg);
    atomicAdd(&a.cnt[1], nsrc);
    atomicAdd(&a.cnt[2], nsnk);
    atomicAdd(&a.cnt[3], dsum);
    wg_sum(s0, sh);  // its barriers also publish cls
    double rz = s0[0], rr = s0[1];
    const double bb = s0[1], stop2 = a.tol * a.tol * bb;
    int it = 0;
    while (it < a.max_iter && rr > stop2) {
        // q = A p on the free beads (p is zero on the electrode beads)
        double pq[1] = {0.0};
        for (int i = threadIdx.x; i < n; i += NET_CG) {
            double q = 0.0;
            if (a.cls[i] == 0) {
                const int dk = min(a.deg[i], NET_DEG);
                const int *nb = a.nbr + size_t(i) * NET_DEG;
                const double *gi = a.g + size_t(i) * NET_DEG;
                double off = 0.0;
                int k = 0;
                // four edges' index and conductance loads in flight at a time,
                // added in edge order
                for (; k + 4 <= dk; k += 4) {
                    const int j0 = nb[k], j1 = nb[k + 1], j2 = nb[k + 2], j3 = nb[k + 3];
                    const double g0 = gi[k], g1 = gi[k + 1], g2 = gi[k + 2], g3 = gi[k + 3];
                    off += g0 * P[j0];
                    off += g1 * P[j1];
                    off += g2 * P[j2];
                    off += g3 * P[j3];
                }
                for (; k < dk; ++k) off += gi[k] * P[nb[k]];
                q = a.diag[i] * P[i] - off;
            }
            a.q[i] = q;
            pq[0] += P[i] * q;
        }
        wg_sum(pq, sh);
        if (!(pq[0] > 0.0)) break;  // same value in every thread
        const double alpha = rz / pq[0];
        double s1[2] = {0.0, 0.0};
        for (int i = threadIdx.x; i < n; i += NET_CG) {
            if (a.cls[i] != 0) continue;
            const double r = a.r[i] - alpha * a.q[i];
            const double dg = a.diag[i];
            const double z = dg > 0.0 ? r / dg : 0.0;
            a.V[i] += alpha * P[i];
            a.r[i] = r;
            a.z[i] = z;
            s1[0] += r * z;
            s1[1] += r * r;
        }
        wg_sum(s1, sh);
        const double beta = rz > 0.0 ? s1[0] / rz : 0.0;
        rz = s1[0];
        rr = s1[1];
        for (int i = threadIdx.x; i < n; i += NET_CG)
            if (a.cls[i] == 0) P[i] = a.z[i] + beta * P[i];
        __syncthreads();  // the next product reads every bead's p
        ++it;
    }
    __syncthreads();  // every potential written
    // Eq. 15 and the current leaving the source electrode
    double st[1] = {0.0};
    for (int i = threadIdx.x; i < n; i += NET_CG) {
        const int ci = a.cls[i];
        const int dk = min(a.deg[i], NET_DEG);
        const double Vi = a.V[i];
        double s = 0.0;
        for (int k = 0; k < dk; ++k) {
            const int j = a.nbr[size_t(i) * NET_DEG + k];
            const double e = a.g[size_t(i) * NET_DEG + k] * (Vi - a.V[j]);
            s += fabs(e);
            if (ci == 1 && a.cls[j] != 1) st[0] += e;
        }
        a.I[i] = 0.5 * s;
    }
    wg_sum(st, sh);
    if (threadIdx.x == 0) {
        a.out[0] = st[0];
        a.out[1] = bb > 0.0 ? sqrt(rr / bb) : 0.0;
        a.out[2] = double(it);
    }
}

// bead j of rod r: X + t e, t from -h to +h in nb - 1 equal steps
__global__ void rod_beads_kernel(const double *rods, int n_rods, int nb, double half, double *pos) {
    const int t = blockIdx.x * blockDim.x + int(threadIdx.x);
    if (t >= n_rods * nb) return;
    const int r = t / nb, j = t - r * nb;
    const double *rod = rods + size_t(r) * ROD_STRIDE;
    const double w = rod[ROD_Q], x = rod[ROD_Q + 1], y = rod[ROD_Q + 2], z = rod[ROD_Q + 3];
    const double e[3] = {2.0 * (x * z + w * y), 2.0 * (y * z - w * x), 1.0 - 2.0 * (x * x + y * y)};
    const double s = -half + 2.0 * half * j / (nb - 1);
#pragma unroll
    for (int d = 0; d < 3; ++d) pos[3 * size_t(t) + d] = rod[ROD_X + d] + s * e[d];
}

}  // namespace

hipError_t launch_net_edges(const NetArgs &a, hipStream_t s) {
    if (a.n <= 0) return hipSuccess;
    const int nblk = (a.n + NET_TB / 64 - 1) / (NET_TB / 64);
    if (a.n <= NET_ROWS) {
        hipLaunchKernelGGL((net_edges_kernel<true, 1>), dim3(nblk), dim3(NET_TB), 0, s, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(net_rows_kernel, dim3(nblk), dim3(NET_TB), 0, s, a);
    } else {
        hipLaunchKernelGGL((net_edges_kernel<false, 4>), dim3((nblk + 3) / 4), dim3(NET_TB), 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_net_solve(const NetArgs &a, hipStream_t s) {
    if (a.n <= 0) return hipSuccess;
    const size_t lds = size_t(a.n) * sizeof(double), lds2 = 2 * lds;
    if (a.n <= NET_CG)
        hipLaunchKernelGGL(net_rows_solve_kernel<1>, dim3(1), dim3(NET_CG), lds2, s, a);
    else if (a.n <= 2 * NET_CG)
        hipLaunchKernelGGL(net_rows_solve_kernel<2>, dim3(1), dim3(NET_CG), lds2, s, a);
    else if (a.n <= 4 * NET_CG)
        hipLaunchKernelGGL(net_rows_solve_kernel<4>, dim3(1), dim3(NET_CG), lds2, s, a);
    else if (a.n <= NET_ROWS)
        hipLaunchKernelGGL(net_rows_solve_kernel<8>, dim3(1), dim3(NET_CG), lds2, s, a);
    else if (a.n <= NET_LDS_P)
        hipLaunchKernelGGL(net_solve_kernel<true>, dim3(1), dim3(NET_CG), lds, s, a);
    else
        hipLaunchKernelGGL(net_solve_kernel<false>, dim3(1), dim3(NET_CG), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_rod_beads(const double *rods, int n_rods, int nb, double half, double *pos, hipStream_t s) {
    const int n = n_rods * nb;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(rod_beads_kernel, dim3((n + 255) / 256), dim3(256), 0, s, rods, n_rods, nb, half, pos);
    return hipGetLastError();
}

}  // namespace lbm
