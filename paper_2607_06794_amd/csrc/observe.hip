// Droplet and deposit observables (gfx950).
//
// Droplet shape: colour C = (rho_A - rho_B) / (rho_A + rho_B) on fluid nodes
// (liquid C > 0).  One thread per (x, y) column scans down from the top for
// the topmost wet node and interpolates the C = 0 crossing above it (column
// height above the wall surface z = 1/2); the droplet height is the largest
// column height.  The footprint half-lengths are the runs of C > 0 on the
// first fluid plane through the given centre, ends interpolated at C = 0, and
// the contact angles follow from the spherical-cap relation
// theta = 2 atan(h / r) (Results, drying dynamics: h, r_x, r_y, theta_x,
// theta_y; the paper leaves the extraction open).
//
// Deposit statistics of the rods (Methods, structural characterisation):
// beads evenly spaced along each axis segment and the segments between them;
// g^b (Eq. 14) = bead count over the mean bead count per bin, S_x^b (Eq. 13)
// = mean of 2 cos^2(zeta) - 1 over the segments whose midpoints fall in the
// bin; axial profiles bin x inside a central strip in y, transverse profiles
// bin y inside a central strip in x.  The sums of a bin have a fixed order, so
// they are deterministic.
//
// Contact graph (Methods, electrical network model): rods connect when their
// axis segments are closer than r_c; clusters by minimum-label propagation
// over an adjacency bitmap (labels converge to the smallest rod index of each
// cluster); a cluster spans when it reaches both x < x_src and x > x_snk.
#include <math.h>

#include "lbm_device.h"
#include "lbm_internal.h"

namespace lbm {

namespace {

template <class S>
__device__ inline double colour_at(const S *f, int64_t fs, const uint8_t *mat, int64_t n, double r0, double r1) {
    const uint8_t m = mat[n] & MAT_ID_MASK;
    double rho[2];
    const double rr[2] = {r0, r1};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < Q; ++i) s += double(Codec<S>::dec(f[(k * Q + i) * fs + n])) + wgt<double>(i) * rr[k];
        rho[k] = s;
    }
    const double tot = rho[0] + rho[1];
    return m == MAT_FLUID && tot > 0.0 ? (rho[0] - rho[1]) / tot : NAN;
}

// A work-group scans COL_X columns, each split over COL_Z threads along z: a
// thread takes one run of planes from the top down, and the first thread of a
// column joins the runs (the colour above a run's top node is the lowest one
// of the run above).  Bound by reading the populations once, in runs of 64
// nodes; one thread per column left a 256 x 128 x 64 lattice with 512
// wavefronts (105 -> 84 us; 128 columns of 8 runs 137, 32 of 32 runs 91).
constexpr int COL_X = 64, COL_Z = 16;  // the joining wavefront: COL_X lanes

template <class S>
__global__ void __launch_bounds__(COL_X * COL_Z) column_height_kernel(ObsArgs o, const S *f) {
    __shared__ double top_c[COL_Z][COL_X], top_above[COL_Z][COL_X], low_c[COL_Z][COL_X];
    __shared__ int top_z[COL_Z][COL_X], wet_n[COL_Z][COL_X];
    const int64_t ncol = int64_t(o.nx) * o.ny;
    const int lx = threadIdx.x % COL_X, seg = threadIdx.x / COL_X;  // seg 0 lowest
    const int64_t c = blockIdx.x * int64_t(COL_X) + lx;
    const int len = (o.nz + COL_Z - 1) / COL_Z, z0 = seg * len, z1 = min(z0 + len, o.nz);
    if (c < ncol) {
        const int x = int(c % o.nx), y = int(c / o.nx);
        double above = NAN, tc = 0.0, ta = NAN;
        int wet = 0, tz = -1;
        for (int z = z1 - 1; z >= z0; --z) {
            const double cz = colour_at(f, o.fs, o.mat, int64_t(z) * ncol + c, o.rho_ref[0], o.rho_ref[1]);
            if (cz > 0.0) {
                ++wet;
                if (tz < 0 && z >= 1) {
                    tz = z;
                    tc = cz;
                    ta = above;
                }
            }
            above = cz;
            if (z == 1) {
                if (y == o.iy) o.line_x[x] = cz;
                if (x == o.ix) o.line_y[y] = cz;
            }
        }
        top_z[seg][lx] = tz;
        top_c[seg][lx] = tc;
        top_above[seg][lx] = ta;
        low_c[seg][lx] = above;
        wet_n[seg][lx] = wet;
    }
    __syncthreads();
    if (seg != 0) return;  // the first wavefront joins the runs and the columns
    double h = 0.0;
    int wet = 0;
    if (c < ncol) {
        for (int q = COL_Z - 1; q >= 0; --q) wet += wet_n[q][lx];
        for (int q = COL_Z - 1; q >= 0; --q) {
            const int z = top_z[q][lx];
            if (z < 0) continue;
            const double cz = top_c[q][lx];
            // the run's own top node: the node above is the next run's lowest
            const double above = z == min((q + 1) * len, o.nz) - 1 ? (z + 1 < o.nz ? low_c[q + 1][lx] : NAN)
                                                                   : top_above[q][lx];
            const double frac = (z + 1 < o.nz && !isnan(above)) ? cz / (cz - above) : 0.5;
            h = (double(z) + frac) - 0.5;
            break;
        }
    }
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
        h = fmax(h, __shfl_xor(h, s, 64));
        wet += __shfl_xor(wet, s, 64);
    }
    if (lx == 0) {
        o.col_h[blockIdx.x] = h;
        o.col_wet[blockIdx.x] = wet;
    }
}

// half-length of the run of wet values through the centre; every thread of the
// work-group calls it and looks for the run's ends in its share of the line
__device__ double run_half_length(const double *line, int n, int centre, int *ends) {
    if (threadIdx.x == 0) {
        ends[0] = -1;  // the last dry value before the centre, the first after
        ends[1] = n;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x)
        if (!(line[i] > 0.0)) {
            if (i <= centre) atomicMax(&ends[0], i);
            if (i >= centre) atomicMin(&ends[1], i);
        }
    __syncthreads();
    const int lo = ends[0] + 1, hi = ends[1] - 1;
    if (lo > centre) return 0.0;  // the centre itself is dry
    double left = lo - 0.5, right = hi + 0.5;
    if (lo - 1 >= 0 && !isnan(line[lo - 1])) left = lo - line[lo] / (line[lo] - line[lo - 1]);
    if (hi + 1 < n && !isnan(line[hi + 1])) right = hi + line[hi] / (line[hi] - line[hi + 1]);
    return 0.5 * (right - left);
}

__global__ void __launch_bounds__(256) shape_final_kernel(ObsArgs o, int nblk) {
    __shared__ double smax[4];
    __shared__ long long swet[4];
    __shared__ int ends[2][2];
    double hm = 0.0;
    long long wet = 0;
    for (int c = threadIdx.x; c < nblk; c += blockDim.x) {
        hm = fmax(hm, o.col_h[c]);
        wet += o.col_wet[c];
    }
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
        hm = fmax(hm, __shfl_xor(hm, s, 64));
        wet += __shfl_xor(wet, s, 64);
    }
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    if (l == 0) {
        smax[w] = hm;
        swet[w] = wet;
    }
    const double rx = run_half_length(o.line_x, o.nx, o.ix, ends[0]);
    const double ry = run_half_length(o.line_y, o.ny, o.iy, ends[1]);
    if (threadIdx.x == 0) {
        for (int q = 1; q < int(blockDim.x >> 6); ++q) {
            hm = fmax(hm, smax[q]);
            wet += swet[q];
        }
        o.out[0] = hm;
        o.out[1] = rx;
        o.out[2] = ry;
        o.out[3] = rx > 0.0 ? 2.0 * atan2(hm, rx) : 0.0;
        o.out[4] = ry > 0.0 ? 2.0 * atan2(hm, ry) : 0.0;
        o.out[5] = double(wet);
    }
}

// ---------------------------------------------------------------------------
// deposit profiles
// ---------------------------------------------------------------------------
__device__ inline double min_img1(double d, double box, int per) { return per ? d - box * rint(d / box) : d; }
__device__ inline double wrap1d(double v, double n) { return v - n * floor(v / n); }
__device__ inline int bin_of(double v, double n, int nb) {
    const int b = int(floor(wrap1d(v, n) * nb / n));
    return b < nb - 1 ? b : nb - 1;
}
__device__ inline void rod_axis(const double *q, double e[3]) {
    const double w = q[0], x = q[1], y = q[2], z = q[3];
    e[0] = 2.0 * (x * z + w * y);
    e[1] = 2.0 * (y * z - w * x);
    e[2] = 1.0 - 2.0 * (x * x + y * y);
}

// One work-group per bin (axial bins first, then transverse): its threads go
// over every bead and the segment before it, a fixed share each, and the sums
// are added in a fixed order.  (One work-group binned rod by rod and then
// added bin by bin in index order: 870 us for 300 rods and 24 bins, now 14.)
constexpr int DEP_TB = 256;

__global__ void __launch_bounds__(DEP_TB) deposit_kernel(DepArgs d) {
    __shared__ double sh_s[DEP_TB / 64];
    __shared__ int sh_n[DEP_TB / 64][2];
    const double nx = d.nx, ny = d.ny;
    const bool axial = int(blockIdx.x) < d.nbx;
    const int b = axial ? blockIdx.x : blockIdx.x - d.nbx;
    // the bin of p along the profile's direction, -1 outside its strip
    auto bin_at = [&](const double p[3]) {
        const bool in = axial ? fabs(min_img1(p[1] - d.yc, ny, d.py)) <= 0.5 * d.strip_y
                              : fabs(min_img1(p[0] - d.xc, nx, d.px)) <= 0.5 * d.strip_x;
        return in ? (axial ? bin_of(p[0], nx, d.nbx) : bin_of(p[1], ny, d.nby)) : -1;
    };
    int cnt = 0, nseg = 0;
    double ssum = 0.0;
    for (int t = threadIdx.x; t < d.n_rods * d.nb; t += DEP_TB) {
        const int r = t / d.nb, j = t - r * d.nb;
        const double *rod = d.rods + r * ROD_STRIDE;
        double e[3];
        rod_axis(rod + ROD_Q, e);
        double X[3] = {rod[ROD_X], rod[ROD_X + 1], rod[ROD_X + 2]};
        // mirror image at the droplet centre (the rod is symmetric end to end)
        if (d.mirror_x) {
            X[0] = 2.0 * d.xc - X[0];
            e[0] = -e[0];
        }
        if (d.mirror_y) {
            X[1] = 2.0 * d.yc - X[1];
            e[1] = -e[1];
        }
        const double tj = -d.half + 2.0 * d.half * j / (d.nb - 1);
        const double p[3] = {X[0] + tj * e[0], X[1] + tj * e[1], X[2] + tj * e[2]};
        cnt += bin_at(p) == b;
        if (j > 0) {
            const double ti = -d.half + 2.0 * d.half * (j - 1) / (d.nb - 1);
            const double prev[3] = {X[0] + ti * e[0], X[1] + ti * e[1], X[2] + ti * e[2]};
            const double m[3] = {0.5 * (prev[0] + p[0]), 0.5 * (prev[1] + p[1]), 0.5 * (prev[2] + p[2])};
            if (bin_at(m) == b) {
                ssum += 2.0 * e[0] * e[0] - 1.0;
                ++nseg;
            }
        }
    }
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
        ssum += __shfl_xor(ssum, s, 64);
        cnt += __shfl_xor(cnt, s, 64);
        nseg += __shfl_xor(nseg, s, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        sh_s[threadIdx.x >> 6] = ssum;
        sh_n[threadIdx.x >> 6][0] = cnt;
        sh_n[threadIdx.x >> 6][1] = nseg;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < DEP_TB / 64; ++w) {
            ssum += sh_s[w];
            cnt += sh_n[w][0];
            nseg += sh_n[w][1];
        }
        double *out = d.out + (axial ? 0 : 3 * DEP_MAXBIN);
        out[b] = double(cnt);
        out[DEP_MAXBIN + b] = nseg > 0 ? ssum / double(nseg) : 0.0;
        out[2 * DEP_MAXBIN + b] = double(nseg);
    }
}

// ---------------------------------------------------------------------------
// contact graph
// ---------------------------------------------------------------------------
struct v3 {
    double x, y, z;
};
__device__ inline v3 operator+(v3 a, v3 b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ inline v3 operator-(v3 a, v3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ inline v3 operator*(double s, v3 a) { return {s * a.x, s * a.y, s * a.z}; }
__device__ inline double vdot(v3 a, v3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }

// distance between segments [p1, q1], [p2, q2]: the stationary point of the
// squared distance if interior, else the best clamped edge
__device__ double seg_dist(v3 p1, v3 q1, v3 p2, v3 q2) {
    const v3 d1 = q1 - p1, d2 = q2 - p2, r = p1 - p2;
    const double a = vdot(d1, d1), e = vdot(d2, d2), f = vdot(d2, r), c = vdot(d1, r), b = vdot(d1, d2);
    double best = 1e300;
    auto tryst = [&](double s, double t) {
        const v3 dd = (p1 + s * d1) - (p2 + t * d2);
        best = fmin(best, sqrt(vdot(dd, dd)));
    };
    const double den = a * e - b * b;
    if (den > 1e-14 * fmax(a * e, 1e-300)) {
        const double s = (b * f - c * e) / den, t = (a * f - b * c) / den;
        if (s >= 0.0 && s <= 1.0 && t >= 0.0 && t <= 1.0) tryst(s, t);
    }
    for (int k = 0; k < 2; ++k) tryst(k, e == 0.0 ? 0.0 : fmin(fmax((b * k + f) / e, 0.0), 1.0));
    for (int k = 0; k < 2; ++k) tryst(a == 0.0 ? 0.0 : fmin(fmax((b * k - c) / a, 0.0), 1.0), k);
    return best;
}

constexpr int ADJ_W = LB_MAX_RODS / 64;

// adjacency rows: one wavefront per rod a, its lanes over the rods b; a pair's
// distance is taken from the lower rod on both of its rows
__global__ void __launch_bounds__(64) graph_rows_kernel(DepArgs d) {
    const int a = blockIdx.x, lane = threadIdx.x;
    const double box[3] = {double(d.nx), double(d.ny), double(d.nz)};
    const int per[3] = {d.px, d.py, d.pz};
    for (int w = 0; w < ADJ_W; ++w) {
        const int b = w * 64 + lane;
        bool join = false;
        if (b < d.n_rods && b != a) {
            const double *ra = d.rods + min(a, b) * ROD_STRIDE, *rb = d.rods + max(a, b) * ROD_STRIDE;
            double ea[3], eb[3];
            rod_axis(ra + ROD_Q, ea);
            rod_axis(rb + ROD_Q, eb);
            const v3 Xa = {ra[ROD_X], ra[ROD_X + 1], ra[ROD_X + 2]}, Ea = {ea[0], ea[1], ea[2]};
            const v3 pa = Xa - d.half * Ea, qa = Xa + d.half * Ea;
            const double dx[3] = {min_img1(rb[ROD_X] - ra[ROD_X], box[0], per[0]),
                                  min_img1(rb[ROD_X + 1] - ra[ROD_X + 1], box[1], per[1]),
                                  min_img1(rb[ROD_X + 2] - ra[ROD_X + 2], box[2], per[2])};
            const v3 Xb = Xa + v3{dx[0], dx[1], dx[2]}, Eb = {eb[0], eb[1], eb[2]};
            join = seg_dist(pa, qa, Xb - d.half * Eb, Xb + d.half * Eb) < d.r_contact;
        }
        const unsigned long long m = __ballot(join);
        if (lane == 0) d.adj[size_t(a) * ADJ_W + w] = m;
    }
}

// clusters from the adjacency rows: every label falls to the smallest rod
// index of its cluster, by the neighbours' labels and by the label's own label
// (pair distances and the clusters' ends by one work-group: 407 -> 33 us)
__global__ void __launch_bounds__(LB_MAX_RODS) graph_kernel(DepArgs d) {
    __shared__ int lab[2][LB_MAX_RODS];
    __shared__ int size[LB_MAX_RODS], ends[LB_MAX_RODS];
    __shared__ int edges, largest, spanning;
    __shared__ int changed[2];
    const int n = d.n_rods, a = threadIdx.x;
    unsigned long long adj[ADJ_W];
#pragma unroll
    for (int w = 0; w < ADJ_W; ++w) adj[w] = a < n ? d.adj[size_t(a) * ADJ_W + w] : 0ull;
    lab[0][a] = a;
    size[a] = ends[a] = 0;
    if (a == 0) edges = largest = spanning = changed[0] = changed[1] = 0;
    __syncthreads();
    // the change flag is double buffered so that every thread reads the same
    // value before it is reset
    int cur = 0;
    for (int it = 0; it <= n; ++it) {
        const int par = it & 1;
        int m = lab[cur][a];
        m = min(m, lab[cur][m]);
#pragma unroll
        for (int w = 0; w < ADJ_W; ++w) {
            unsigned long long bits = adj[w];
            while (bits) {
                const int b = w * 64 + __builtin_ctzll(bits);
                bits &= bits - 1;
                m = min(m, lab[cur][b]);
            }
        }
        lab[cur ^ 1][a] = m;
        if (m != lab[cur][a]) changed[par] = 1;
        __syncthreads();
        const bool go = changed[par] != 0;
        if (a == 0) changed[par ^ 1] = 0;
        __syncthreads();
        cur ^= 1;
        if (!go) break;
    }
    if (a < n) {
        int deg = 0;
#pragma unroll
        for (int w = 0; w < ADJ_W; ++w) deg += __popcll(adj[w]);
        atomicAdd(&edges, deg);
        const int l = lab[cur][a];
        atomicAdd(&size[l], 1);
        // a cluster spans when rods of it reach both sides
        const double *ra = d.rods + a * ROD_STRIDE;
        double ea[3];
        rod_axis(ra + ROD_Q, ea);
        const double reach = d.half * fabs(ea[0]);
        const int side = (ra[ROD_X] - reach < d.x_src ? 1 : 0) | (ra[ROD_X] + reach > d.x_snk ? 2 : 0);
        if (side) atomicOr(&ends[l], side);
        d.labels[a] = l;
    }
    __syncthreads();
    atomicMax(&largest, size[a]);
    if (ends[a] == 3) spanning = 1;
    __syncthreads();
    if (a == 0) {
        d.graph[0] = n;
        d.graph[1] = edges / 2;
        d.graph[2] = largest;
        d.graph[3] = spanning;
    }
}

__global__ void rod_map_kernel(const uint8_t *mat, int nx, int ny, int nz, int32_t *map) {
    const int64_t ncol = int64_t(nx) * ny;
    for (int64_t c = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; c < ncol; c += int64_t(gridDim.x) * blockDim.x) {
        int cnt = 0;
        for (int z = 0; z < nz; ++z) cnt += (mat[int64_t(z) * ncol + c] & MAT_ID_MASK) == MAT_ROD;
        map[c] = cnt;
    }
}

int grid_cols(int64_t ncol) {
    const int64_t g = (ncol + 255) / 256;
    return int(g < 1 ? 1 : (g > 4096 ? 4096 : g));
}

}  // namespace

// Shan-Chen equation of state at probe nodes: p = c_s^2 (rho_A + rho_B) +
// G c_s^2 psi_A psi_B with psi = rho on fluid nodes; NaN at non-fluid probes
template <class S>
__global__ void pressure_probe_kernel(const S *f, int64_t fs, const uint8_t *mat, int nx, int ny, int nz, double r0,
                                      double r1, double G, const int *xyz, int n, double *out) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const int x = xyz[3 * q], y = xyz[3 * q + 1], z = xyz[3 * q + 2];
    const int64_t node = (int64_t(z) * ny + y) * nx + x;
    if ((mat[node] & MAT_ID_MASK) != MAT_FLUID) {
        out[q] = __builtin_nan("");
        return;
    }
    const double rr[2] = {r0, r1};
    double rho[2];
    for (int k = 0; k < 2; ++k) {
        double s = 0.0;
        for (int i = 0; i < Q; ++i) s += double(Codec<S>::dec(f[(k * Q + i) * fs + node])) + wgt<double>(i) * rr[k];
        rho[k] = s;
    }
    out[q] = (rho[0] + rho[1]) / 3.0 + G / 3.0 * rho[0] * rho[1];
}

hipError_t launch_droplet(int prec, const void *f, const ObsArgs &o, hipStream_t s) {
    const dim3 grid(unsigned((int64_t(o.nx) * o.ny + COL_X - 1) / COL_X));
    hipError_t e;
    switch (prec) {
        case LB_F64:
            hipLaunchKernelGGL(column_height_kernel<double>, grid, dim3(COL_X * COL_Z), 0, s, o,
                               static_cast<const double *>(f));
            break;
        case LB_F32:
            hipLaunchKernelGGL(column_height_kernel<float>, grid, dim3(COL_X * COL_Z), 0, s, o,
                               static_cast<const float *>(f));
            break;
        case LB_F16DEV:
            hipLaunchKernelGGL(column_height_kernel<_Float16>, grid, dim3(COL_X * COL_Z), 0, s, o,
                               static_cast<const _Float16 *>(f));
            break;
        case LB_BF16DEV:
            hipLaunchKernelGGL(column_height_kernel<bf16_t>, grid, dim3(COL_X * COL_Z), 0, s, o,
                               static_cast<const bf16_t *>(f));
            break;
        default:
            return hipErrorInvalidValue;
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(shape_final_kernel, dim3(1), dim3(256), 0, s, o, int(grid.x));
    return hipGetLastError();
}

// one image's profiles into the ensemble sums: Eq. 14 normalises the bead
// counts by their mean over the bins (summed in bin order by one thread);
// Eq. 13's bin means enter only where the image has segments
__global__ void __launch_bounds__(2 * DEP_MAXBIN) deposit_accumulate_kernel(const double *out, int nbx, int nby,
                                                                           double *acc) {
    __shared__ double mean[2];
    if (threadIdx.x < 2) {
        const int d = threadIdx.x, nb = d ? nby : nbx;
        const double *cnt = out + d * 3 * DEP_MAXBIN;
        double t = 0.0;
        for (int b = 0; b < nb; ++b) t += cnt[b];
        mean[d] = t / nb;
    }
    __syncthreads();
    const int d = threadIdx.x >= DEP_MAXBIN, b = threadIdx.x - d * DEP_MAXBIN;
    if (b >= (d ? nby : nbx)) return;
    const double *o = out + d * 3 * DEP_MAXBIN;
    const double nseg = o[2 * DEP_MAXBIN + b];
    acc[d * DEP_MAXBIN + b] += mean[d] > 0.0 ? o[b] / mean[d] : 0.0;
    acc[(2 + d) * DEP_MAXBIN + b] += nseg > 0.0 ? o[DEP_MAXBIN + b] : 0.0;
    acc[(4 + d) * DEP_MAXBIN + b] += nseg > 0.0 ? 1.0 : 0.0;
    acc[(6 + d) * DEP_MAXBIN + b] += nseg;
}

__global__ void __launch_bounds__(2 * DEP_MAXBIN) deposit_finish_kernel(const double *acc, int nbx, int nby,
                                                                       int images, double *out) {
    const int d = threadIdx.x >= DEP_MAXBIN, b = threadIdx.x - d * DEP_MAXBIN;
    if (b >= (d ? nby : nbx)) return;
    const double c = acc[(4 + d) * DEP_MAXBIN + b];
    double *o = out + d * 3 * DEP_MAXBIN;
    o[b] = acc[d * DEP_MAXBIN + b] / images;
    o[DEP_MAXBIN + b] = c > 0.0 ? acc[(2 + d) * DEP_MAXBIN + b] / c : 0.0;
    o[2 * DEP_MAXBIN + b] = acc[(6 + d) * DEP_MAXBIN + b];
}

hipError_t launch_deposit_accumulate(const DepArgs &d, double *acc, hipStream_t s) {
    hipLaunchKernelGGL(deposit_kernel, dim3(d.nbx + d.nby), dim3(DEP_TB), 0, s, d);
    hipLaunchKernelGGL(deposit_accumulate_kernel, dim3(1), dim3(2 * DEP_MAXBIN), 0, s, d.out, d.nbx, d.nby, acc);
    return hipGetLastError();
}

hipError_t launch_deposit_finish(const double *acc, int nbx, int nby, int images, double *out, hipStream_t s) {
    hipLaunchKernelGGL(deposit_finish_kernel, dim3(1), dim3(2 * DEP_MAXBIN), 0, s, acc, nbx, nby, images, out);
    return hipGetLastError();
}

hipError_t launch_deposit(const DepArgs &d, hipStream_t s) {
    hipLaunchKernelGGL(deposit_kernel, dim3(d.nbx + d.nby), dim3(DEP_TB), 0, s, d);
    if (d.n_rods > 0) hipLaunchKernelGGL(graph_rows_kernel, dim3(d.n_rods), dim3(64), 0, s, d);
    hipLaunchKernelGGL(graph_kernel, dim3(1), dim3(LB_MAX_RODS), 0, s, d);
    return hipGetLastError();
}

hipError_t launch_rod_map(const uint8_t *mat, int nx, int ny, int nz, int32_t *map, hipStream_t s) {
    hipLaunchKernelGGL(rod_map_kernel, dim3(grid_cols(int64_t(nx) * ny)), dim3(256), 0, s, mat, nx, ny, nz, map);
    return hipGetLastError();
}

hipError_t launch_pressure(int prec, const void *f, int64_t fs, const uint8_t *mat, int nx, int ny, int nz,
                           const double rref[2], double G, const int *xyz, int n, double *out, hipStream_t s) {
    const dim3 grid((n + 255) / 256);
    switch (prec) {
        case LB_F64:
            hipLaunchKernelGGL(pressure_probe_kernel<double>, grid, dim3(256), 0, s, static_cast<const double *>(f), fs,
                               mat, nx, ny, nz, rref[0], rref[1], G, xyz, n, out);
            break;
        case LB_F32:
            hipLaunchKernelGGL(pressure_probe_kernel<float>, grid, dim3(256), 0, s, static_cast<const float *>(f), fs, mat,
                               nx, ny, nz, rref[0], rref[1], G, xyz, n, out);
            break;
        case LB_F16DEV:
            hipLaunchKernelGGL(pressure_probe_kernel<_Float16>, grid, dim3(256), 0, s, static_cast<const _Float16 *>(f),
                               fs, mat, nx, ny, nz, rref[0], rref[1], G, xyz, n, out);
            break;
        case LB_BF16DEV:
            hipLaunchKernelGGL(pressure_probe_kernel<bf16_t>, grid, dim3(256), 0, s, static_cast<const bf16_t *>(f), fs,
                               mat, nx, ny, nz, rref[0], rref[1], G, xyz, n, out);
            break;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace lbm
