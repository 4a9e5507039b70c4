// Learned surrogate (gfx950): restriction of the lattice state to a coarse
// canvas, prolongation and lift back to populations, and the training and
// inference kernels of a 3-D convolutional U-Net.
//
// Convolutions are implicit GEMMs on BF16 MFMA (32 x 32 x 16, FP32
// accumulation).  Tensors are channels-last, [D][H][W][C], C a multiple of 8.
//   forward  y[p, o]  = b[o] + sum_{t, c} x[p + o_t, c] w[t, c, o]
//            M = positions, N = output channels, K = 27 x input channels
//   dgrad    dx[q, c] = sum_{t, o} g[q - o_t, o] w[t, c, o],  g = dy (y > 0)
//            M = positions, N = input channels, K = 27 x output channels
//   wgrad    dw[t, c, o] += sum_p x[p + o_t, c] g[p, o]
//            M = input channels, N = output channels of one tap, K = positions
// The kernel is chosen by the volume and N (launch_conv): a GEMM over tiles of
// consecutive positions, the same with K cut into parts, bricks of positions that
// share their input halo in LDS, or small bricks whose K is split over the
// wavefronts.
// The decoder's inputs are read in place: channels [0, c1) from the coarser
// level through nearest-neighbour upsampling, [c1, c1 + c2) from the skip.
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <initializer_list>
#include <type_traits>

#include "lbm_device.h"
#include "lbm_internal.h"
#include "node_access.h"

namespace lbm {

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

__device__ inline uint16_t f2bf(float x) {
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest even
    return static_cast<uint16_t>(u >> 16);
}
__device__ inline float bf2f(uint16_t b) { return __uint_as_float(uint32_t(b) << 16); }


// n elements of the input gradient (i < 0: none): FP32, or where the input is a
// ReLU layer's output my, that layer's pre-activation gradient BF16(v (my > 0)) at
// once (instead of FP32 and a pass over it: 9 us per layer of 262 144 x 32).  One
// branch for all of them, and the mask's loads before its first use: a test per
// element cost the GEMM of 262 144 x 96 70 us.
template <int n, class I>
__device__ __forceinline__ void put_grads(const ConvArgs &a, float *dx, const I (&i)[n], const float (&v)[n]) {
    if (a.mg) {
        float m[n];
#pragma unroll
        for (int q = 0; q < n; ++q) m[q] = bf2f(a.my[i[q] < 0 ? I(0) : i[q]]);
#pragma unroll
        for (int q = 0; q < n; ++q)
            if (i[q] >= 0) a.mg[i[q]] = f2bf(m[q] > 0.0f ? v[q] : 0.0f);
    } else {
#pragma unroll
        for (int q = 0; q < n; ++q)
            if (i[q] >= 0) dx[i[q]] = v[q];
    }
}

// ---------------------------------------------------------------------------
// forward and input gradient: one implicit GEMM, C[M][N] = sum_k A[M][k] B[k][N]
//   forward: M = positions p, N = output channels o, k = (tap t, input channel c),
//            A[p][k] = x[p + o_t][c], B[k][o] = wt[o][t][c] (packed weights)
//   dgrad:   M = positions q, N = input channels c, k = (tap t, output channel o),
//            A[q][k] = g[q - o_t][o], B[k][c] = w[t][c][o]
// Both operands sit in LDS K-contiguous per row ([row][BK + 8], 80-byte rows,
// conflict-free 16-byte reads), so every MFMA operand is one 128-bit LDS
// read: lane l takes row l % 32, k = 8 (l / 32) .. + 7 of a 32 x 32 x 16
// block.  K advances by BK = 32 per stage through two LDS buffers; the global
// loads of stage s + 1 are in flight while stage s computes, one barrier per
// stage.  TPR threads share an A row (4 / TPR k-groups of 8 channels each);
// the row's coordinates and its 27-bit mask of in-volume taps are computed
// once, so a stage costs each thread a few integer operations per load.
// ---------------------------------------------------------------------------
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
constexpr int BK = 32, LDK = BK + 8;

// bit t set when tap t of (d, h, w) lies inside the volume
__device__ inline unsigned tap_mask(int d, int h, int w, int D, int H, int W) {
    const unsigned mz = 2u | (d > 0 ? 1u : 0u) | (d < D - 1 ? 4u : 0u);
    const unsigned my = 2u | (h > 0 ? 1u : 0u) | (h < H - 1 ? 4u : 0u);
    const unsigned mx = 2u | (w > 0 ? 1u : 0u) | (w < W - 1 ? 4u : 0u);
    unsigned m = 0;
#pragma unroll
    for (int t = 0; t < 27; ++t)
        if ((mz >> (t / 9)) & (my >> ((t / 3) % 3)) & (mx >> (t % 3)) & 1u) m |= 1u << t;
    return m;
}

template <int BM, int BN, int WM, int WN, bool DGRAD>
__global__ void __launch_bounds__(256) conv_gemm_kernel(ConvArgs a, const uint16_t *g, float *dx) {
    static_assert(WM * WN == 4, "four wavefronts");
    constexpr int MB = BM / WM / 32, NB = BN / WN / 32;
    static_assert(MB >= 1 && NB >= 1 && MB * WM * 32 == BM && NB * WN * 32 == BN, "tile shape");
    constexpr int TPR = 256 / BM, GPT = 4 / TPR;  // threads per A row, k-groups per thread
    constexpr int BLD = BN * 4;                    // B loads (16 bytes) per stage
    constexpr int BLT = BLD >= 256 ? BLD / 256 : 1;
    __shared__ __attribute__((aligned(16))) uint16_t As[2][BM * LDK];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][BN * LDK];

    const int tid = threadIdx.x, wv = tid >> 6, l = tid & 63;
    const int P = a.D * a.H * a.W;
    const int HW = a.H * a.W;
    const int cin = a.c1 + a.c2;
    const int N = DGRAD ? cin : a.cout;   // columns of C
    const int kc = DGRAD ? a.cout : cin;  // channels per tap along k
    const int Kd = 27 * kc;
    const int m0 = blockIdx.x * BM;
    const int n0 = blockIdx.y * BN;
    const int wm = (wv / WN) * MB * 32, wn = (wv % WN) * NB * 32;

    // ---- this thread's A row and its k-groups
    // rows tid % BM; the k-groups (tid / BM) * GPT .. are the same for a whole
    // wavefront, so its tap and channel bookkeeping is scalar
    const int ar = tid % BM, ag0 = __builtin_amdgcn_readfirstlane((tid / BM) * GPT);
    const int p = m0 + ar;
    const bool prow = p < P;
    const int pw = p % a.W, ph = (p / a.W) % a.H, pd = p / HW;
    unsigned tmask = prow ? tap_mask(pd, ph, pw, a.D, a.H, a.W) : 0u;
    int gt[GPT], gc[GPT];  // tap and channel of each k-group at the current stage
#pragma unroll
    for (int j = 0; j < GPT; ++j) {
        gt[j] = 8 * (ag0 + j) / kc;
        gc[j] = 8 * (ag0 + j) % kc;
    }
    const int H2 = a.H >> 1, W2 = a.W >> 1;

    // ---- B: BN rows x 4 k-groups per stage
    int bn[BLT], bgi[BLT], bt[BLT], bc[BLT];
    bool bon[BLT];
#pragma unroll
    for (int j = 0; j < BLT; ++j) {
        const int idx = tid + 256 * j;
        bn[j] = idx >> 2;
        bgi[j] = idx & 3;
        bon[j] = idx < BLD && n0 + bn[j] < N;
        bt[j] = 8 * bgi[j] / kc;
        bc[j] = 8 * bgi[j] % kc;
    }

    // Loads are unconditional (an invalid one reads a safe address) and the
    // zero fill happens at the LDS store, so no load waits on another.
    uint4 ra[GPT], rb[BLT];
    bool aok[GPT], bok[BLT];
    const uint16_t *asafe = DGRAD ? g : a.x1;
    auto load = [&](int k0) {
#pragma unroll
        for (int j = 0; j < GPT; ++j) {
            const int t = gt[j], c = gc[j];
            const bool ok = prow && (k0 + 8 * (ag0 + j) < Kd) && ((tmask >> (DGRAD ? 26 - t : t)) & 1u);
            const int dz = t / 9 - 1, dyy = (t / 3) % 3 - 1, dxx = t % 3 - 1;
            const uint16_t *src;
            if (DGRAD) {
                src = g + (p - (dz * HW + dyy * a.W + dxx)) * a.cout + c;
            } else if (c < a.c1) {
                if (a.up1) {
                    const int q = (((pd + dz) >> 1) * H2 + ((ph + dyy) >> 1)) * W2 + ((pw + dxx) >> 1);
                    src = a.x1 + q * a.c1 + c;
                } else {
                    src = a.x1 + (p + dz * HW + dyy * a.W + dxx) * a.c1 + c;
                }
            } else {
                src = a.x2 + (p + dz * HW + dyy * a.W + dxx) * a.c2 + (c - a.c1);
            }
            ra[j] = *reinterpret_cast<const uint4 *>(ok ? src : asafe);
            aok[j] = ok;
        }
#pragma unroll
        for (int j = 0; j < BLT; ++j) {
            const bool ok = bon[j] && k0 + 8 * bgi[j] < Kd;
            const uint16_t *src = DGRAD ? a.w + (bt[j] * cin + n0 + bn[j]) * a.cout + bc[j]
                                        : a.wt + (n0 + bn[j]) * Kd + k0 + 8 * bgi[j];
            rb[j] = *reinterpret_cast<const uint4 *>(ok ? src : (DGRAD ? a.w : a.wt));
            bok[j] = ok;
        }
    };
    auto advance = [&]() {
#pragma unroll
        for (int j = 0; j < GPT; ++j) {
            gc[j] += BK;
            while (gc[j] >= kc) {
                gc[j] -= kc;
                ++gt[j];
            }
        }
        if (DGRAD) {
#pragma unroll
            for (int j = 0; j < BLT; ++j) {
                bc[j] += BK;
                while (bc[j] >= kc) {
                    bc[j] -= kc;
                    ++bt[j];
                }
            }
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int j = 0; j < GPT; ++j)
            *reinterpret_cast<uint4 *>(&As[buf][ar * LDK + 8 * (ag0 + j)]) = aok[j] ? ra[j] : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < BLT; ++j)
            if (tid + 256 * j < BLD)
                *reinterpret_cast<uint4 *>(&Bs[buf][bn[j] * LDK + 8 * bgi[j]]) = bok[j] ? rb[j] : make_uint4(0, 0, 0, 0);
    };

    v16f acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    const int nst = (Kd + BK - 1) / BK;
    load(0);
    store(0);
    __syncthreads();
    for (int st = 0; st < nst; ++st) {
        const int cur = st & 1;
        if (st + 1 < nst) {
            advance();
            load((st + 1) * BK);
        }
#pragma unroll
        for (int kk = 0; kk < BK; kk += 16) {
            v8bf fa[MB], fb[NB];
#pragma unroll
            for (int i = 0; i < MB; ++i)
                fa[i] = *reinterpret_cast<const v8bf *>(&As[cur][(wm + 32 * i + (l & 31)) * LDK + kk + 8 * (l >> 5)]);
#pragma unroll
            for (int j = 0; j < NB; ++j)
                fb[j] = *reinterpret_cast<const v8bf *>(&Bs[cur][(wn + 32 * j + (l & 31)) * LDK + kk + 8 * (l >> 5)]);
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
        if (st + 1 < nst) store(cur ^ 1);
        __syncthreads();
    }

    // D element e of lane l: row 8 (e / 4) + 4 (l / 32) + e % 4, column l % 32
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int col = n0 + wn + 32 * j + (l & 31);
            if (col >= N) continue;
            const auto row = [&](int e) { return m0 + wm + 32 * i + 8 * (e >> 2) + 4 * (l >> 5) + (e & 3); };
            if constexpr (DGRAD) {
                int at[16];
                float v[16];
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    at[e] = row(e) < P ? row(e) * cin + col : -1;
                    v[e] = acc[i][j][e];
                }
                put_grads(a, dx, at, v);
                continue;
            }
            const float bias = a.b ? a.b[col] : 0.0f;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                if (row(e) >= P) continue;
                float v = acc[i][j][e] + bias;
                if (a.relu) v = fmaxf(v, 0.0f);
                if (a.y) a.y[row(e) * a.cout + col] = f2bf(v);
                if (a.yf) a.yf[row(e) * a.cout + col] = v;
            }
        }
}

// The GEMM with K cut into KS parts inside a work-group, for layers whose tiles do
// not fill the chip: tiles of T x T, four wavefronts per part with LDS buffers of
// their own, the parts' sums met in LDS.  A stage of BK channels lies inside one
// tap and one of the two inputs (channel counts are multiples of BK), so that an
// address costs a few scalars and one addition; rows that a tap takes outside the
// volume read past the buffer's end, which gives zero.  Two stages are in flight.
// The parts are cut and added as conv_small does (shorter ones first, the last
// first among equals): the same sums bit for bit.
//
// Bound by the latency of a stage (0.2 us with three parts, 0.4 for a part alone).
// 29 295 positions, 128 -> 64 channels: 40 us (326 TFLOP/s); 93 for conv_small with
// its two parts, 65 for a GEMM whose parts were work-groups that added with atomics.
template <int T, int KS, bool DG>
__global__ void __launch_bounds__(256 * KS) conv_split_kernel(ConvArgs a, const uint16_t *g, float *dx) {
    constexpr int MB = T / 64, LPT = T / 64;  // blocks of 32 per wavefront and side, rows per thread
    __shared__ __attribute__((aligned(16))) uint16_t lds[KS][2][2 * T * LDK];  // [part][buffer][rows of A, then of B]
    const int part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    const int tid = threadIdx.x & 255, wv = tid >> 6, l = tid & 63;
    const int P = a.D * a.H * a.W, HW = a.H * a.W, cin = a.c1 + a.c2;
    const int N = DG ? cin : a.cout, kc = DG ? a.cout : cin, nst = 27 * kc / BK;
    const int m0 = blockIdx.x * T, n0 = blockIdx.y * T, wm = (wv >> 1) * MB * 32, wn = (wv & 1) * MB * 32;
    const int s0 = nst * part / KS, cnt = nst * (part + 1) / KS - s0;  // this part's stages
    // this thread's rows tid / 4 + 64 j of both tiles, channels 8 (tid % 4) .. + 7
    const int row = tid >> 2, k8 = 8 * (tid & 3), H2 = a.H >> 1, W2 = a.W >> 1;
    int p[LPT], px[LPT], py[LPT], pz[LPT];
    unsigned tmask[LPT];
    uint32_t bo[LPT];
#pragma unroll
    for (int j = 0; j < LPT; ++j) {
        p[j] = m0 + row + 64 * j;
        px[j] = p[j] % a.W;
        py[j] = p[j] / a.W % a.H;
        pz[j] = p[j] / HW;
        tmask[j] = p[j] < P ? tap_mask(pz[j], py[j], px[j], a.D, a.H, a.W) : 0u;
        // columns past the last read its weights and are not stored
        bo[j] = uint32_t(min(n0 + row + 64 * j, N - 1) * (DG ? a.cout : 27 * cin) + k8) * 2u;
    }
    const auto wr = make_rsrc(DG ? a.w : a.wt, uint32_t(27 * cin) * uint32_t(a.cout) * 2u);
    int t = s0 * BK / kc, c = s0 * BK % kc;  // tap and channel of the next stage to load
    struct Stage {
        uint4 a[LPT], b[LPT];
    } in[2];
    const auto load = [&](Stage &r) {
        const int tt = min(t, 26);  // (past the last stage: loaded, not used)
        const int dz = tt / 9 - 1, dy = tt / 3 % 3 - 1, dxx = tt % 3 - 1;
        const bool skip = !DG && c >= a.c1, up = !DG && !skip && a.up1;
        const int C = DG ? a.cout : (skip ? a.c2 : a.c1), cc = skip ? c - a.c1 : c;
        const uint32_t bytes = uint32_t(up ? P >> 3 : P) * uint32_t(C) * 2u;
        const auto xr = make_rsrc(DG ? g : (skip ? a.x2 : a.x1), bytes);
        const uint32_t so = uint32_t(DG ? tt * cin * a.cout + c : tt * cin + c) * 2u;
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
            int q = p[j] + (DG ? -1 : 1) * (dz * HW + dy * a.W + dxx);
            if (up) q = (((pz[j] + dz) >> 1) * H2 + ((py[j] + dy) >> 1)) * W2 + ((px[j] + dxx) >> 1);
            const bool ok = (tmask[j] >> (DG ? 26 - tt : tt)) & 1u;
            const auto va = __builtin_amdgcn_raw_buffer_load_b128(xr, ok ? uint32_t(q * C + cc + k8) * 2u : bytes, 0, 0);
            const auto vb = __builtin_amdgcn_raw_buffer_load_b128(wr, bo[j], so, 0);
            r.a[j] = make_uint4(va[0], va[1], va[2], va[3]);
            r.b[j] = make_uint4(vb[0], vb[1], vb[2], vb[3]);
        }
        c += BK;
        if (c >= kc) {
            c = 0;
            ++t;
        }
    };
    const auto store = [&](const Stage &r, int buf) {
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
            *reinterpret_cast<uint4 *>(&lds[part][buf][(row + 64 * j) * LDK + k8]) = r.a[j];
            *reinterpret_cast<uint4 *>(&lds[part][buf][(T + row + 64 * j) * LDK + k8]) = r.b[j];
        }
    };
    v16f acc[MB][MB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
    // stage st from buffer cur, while the next goes to LDS and the one after is loaded
    const auto stage = [&](int st, int cur, Stage &next, Stage &after) {
        load(after);
        if (st < cnt) {
#pragma unroll
            for (int kk = 0; kk < BK; kk += 16) {
                v8bf fa[MB], fb[MB];
                const uint16_t *at = lds[part][cur] + (l & 31) * LDK + kk + 8 * (l >> 5);
#pragma unroll
                for (int i = 0; i < MB; ++i) {
                    fa[i] = *reinterpret_cast<const v8bf *>(at + (wm + 32 * i) * LDK);
                    fb[i] = *reinterpret_cast<const v8bf *>(at + (T + wn + 32 * i) * LDK);
                }
#pragma unroll
                for (int i = 0; i < MB; ++i)
#pragma unroll
                    for (int j = 0; j < MB; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);  // the wait for the next stage's loads stays behind the products
        store(next, cur ^ 1);
        __syncthreads();
    };
    load(in[0]);
    load(in[1]);
    store(in[0], 0);
    __syncthreads();
    const int most = (nst + KS - 1) / KS;  // the longest part's: every wavefront passes the same barriers
    int st = 0;
    for (; st + 1 < most; st += 2) {
        stage(st, 0, in[1], in[0]);
        stage(st + 1, 1, in[0], in[1]);
    }
    if (st < most) stage(st, 0, in[1], in[0]);

    // the parts in the order in which they are added
    const auto len = [&](int z) { return nst * (z + 1) / KS - nst * z / KS; };
    int order[KS];
#pragma unroll
    for (int q = 0; q < KS; ++q) {
        int rank = 0;
#pragma unroll
        for (int z = 0; z < KS; ++z) rank += len(z) < len(q) || (len(z) == len(q) && z > q);
#pragma unroll
        for (int r = 0; r < KS; ++r)
            if (rank == r) order[r] = q;
    }
    // first part's wavefronts: its own sums and the others', from LDS
    float *sum = reinterpret_cast<float *>(lds);  // [part - 1][block column][element][thread]
    static_assert((KS - 1) * MB * 4096 * 4 <= sizeof(lds), "the parts' sums fit");
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        if (part > 0) {
#pragma unroll
            for (int j = 0; j < MB; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) sum[((part - 1) * MB + j) * 4096 + e * 256 + tid] = acc[i][j][e];
        }
        __syncthreads();
        if (part == 0) {
#pragma unroll
            for (int j = 0; j < MB; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    float v = 0.0f;
#pragma unroll
                    for (int r = 0; r < KS; ++r)
                        v += order[r] == 0 ? acc[i][j][e] : sum[((order[r] - 1) * MB + j) * 4096 + e * 256 + tid];
                    acc[i][j][e] = v;
                }
        }
        if (i + 1 < MB) __syncthreads();
    }
    if (part > 0) return;

    // D element e of lane l: row 8 (e / 4) + 4 (l / 32) + e % 4, column l % 32
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            const int col = n0 + wn + 32 * j + (l & 31);
            if (col >= N) continue;
            int at[16];
            float v[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int r = m0 + wm + 32 * i + 8 * (e >> 2) + 4 * (l >> 5) + (e & 3);
                at[e] = r < P ? r * N + col : -1;
                v[e] = acc[i][j][e];
            }
            if constexpr (DG) {
                put_grads(a, dx, at, v);
                continue;
            }
            const float bias = a.b ? a.b[col] : 0.0f;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                if (at[e] < 0) continue;
                float r = v[e] + bias;
                if (a.relu) r = fmaxf(r, 0.0f);
                if (a.y) a.y[at[e]] = f2bf(r);
                if (a.yf) a.yf[at[e]] = r;
            }
        }
}

// Forward convolution of a brick of ZB x 8 x 8 positions (M = 64 ZB rows)
// against up to 32 WN output channels, for volumes made of whole bricks:
// ZB = 4, WN = 1 for layers of up to 32 output channels, ZB = 2, WN = 2 for
// up to 64.  Per chunk of 32 input channels the brick's (ZB + 2) x 10 x 10
// input halo is staged in LDS once, the weights nine taps at a time; every
// tap's A operand is then the halo read at the tap's offset, so each input
// element leaves L2 a few times instead of 27.  Each wavefront owns 64 rows
// (two 32-row MFMA blocks) of one 32-column block.  Summation order: chunk,
// tap, channel.
constexpr int BRY = 8, BRX = 8, HLY = BRY + 2, HLX = BRX + 2;
constexpr int BR_TG = 9;  // taps per weight stage (one dz plane of taps)

template <int ZB, int WN>
struct Brick {
    static constexpr int BN = 32 * WN;
    static constexpr int NHALO = (ZB + 2) * HLY * HLX;
    static constexpr int HL = (NHALO * 4 + 255) / 256;          // halo loads per thread
    static constexpr int WE = BR_TG * BN * 4;                   // 16-byte weight elements per stage
    static constexpr int WL = (WE + 255) / 256;                 // weight loads per thread
    static_assert(64 * ZB * WN == 256, "four wavefronts of 64 rows x 32 columns");
};

// per-component select (a select between two uint4 values is lowered to a
// load through a selected address with the zero kept in scratch)
__device__ __forceinline__ uint4 keep4(bool ok, uint4 v) {
    return make_uint4(ok ? v.x : 0u, ok ? v.y : 0u, ok ? v.z : 0u, ok ? v.w : 0u);
}

// loads of a brick's input halo for channels c0 .. c0 + 31 into registers;
// an invalid element loads a safe address and becomes zero
template <int ZB, int WN, bool DG>
__device__ __forceinline__ void brick_fetch_halo(const ConvArgs &a, const uint16_t *g, int tid, int x0, int y0,
                                                 int z0, int c0, uint4 (&hv)[Brick<ZB, WN>::HL]) {
    using B = Brick<ZB, WN>;
    const int cin = DG ? a.cout : a.c1 + a.c2;  // channels of the staged input
    const int H2 = a.H >> 1, W2 = a.W >> 1;
#pragma unroll
    for (int j = 0; j < B::HL; ++j) {
        const int e = tid + 256 * j;
        const int hp = e >> 2, gi = e & 3;
        const int hz = hp / (HLY * HLX), hy = (hp / HLX) % HLY, hx = hp % HLX;
        const int z = z0 + hz - 1, y = y0 + hy - 1, x = x0 + hx - 1;
        const int c = c0 + 8 * gi;
        const bool ok = e < B::NHALO * 4 && z >= 0 && z < a.D && y >= 0 && y < a.H && x >= 0 && x < a.W && c < cin;
        const uint16_t *src = DG ? g : a.x1;
        if (ok && DG) {
            src = g + int64_t(z * a.H + y) * a.W * a.cout + int64_t(x) * a.cout + c;
        } else if (ok) {
            if (c < a.c1)
                src = a.up1 ? a.x1 + (int64_t((z >> 1) * H2 + (y >> 1)) * W2 + (x >> 1)) * a.c1 + c
                            : a.x1 + (int64_t(z * a.H + y) * a.W + x) * a.c1 + c;
            else
                src = a.x2 + (int64_t(z * a.H + y) * a.W + x) * a.c2 + (c - a.c1);
        }
        hv[j] = keep4(ok, *reinterpret_cast<const uint4 *>(src));
    }
}

// loads of the weights of taps t0 .. t0 + 8 for channels c0 .. c0 + 31
// forward: B[n = output channel][k = input channel] = wt[n][t][c]
// input gradient: B[n = input channel][k = output channel] = w[t][n][k]
template <int ZB, int WN, bool DG>
__device__ __forceinline__ void brick_fetch_w(const ConvArgs &a, int tid, int c0, int t0,
                                              uint4 (&wr)[Brick<ZB, WN>::WL]) {
    using B = Brick<ZB, WN>;
    const int cin = a.c1 + a.c2, Kd = 27 * cin;
    const int kc = DG ? a.cout : cin, nn = DG ? cin : a.cout;
#pragma unroll
    for (int j = 0; j < B::WL; ++j) {
        const int e = tid + 256 * j;
        const int t = t0 + e / (B::BN * 4), n = (e >> 2) % B::BN, gi = e & 3;
        const int c = c0 + 8 * gi;
        const bool ok = e < B::WE && n < nn && c < kc;
        const uint16_t *src = DG ? a.w + (int64_t(t) * cin + n) * a.cout + c : a.wt + int64_t(n) * Kd + t * cin + c;
        wr[j] = keep4(ok, *reinterpret_cast<const uint4 *>(ok ? src : (DG ? a.w : a.wt)));
    }
}

// DG: the input gradient dx[q][c] = sum_{t, o} g[q - o_t][o] w[t][c][o], the
// same computation over g with the taps mirrored, dx stored in FP32
template <int ZB, int WN, bool DG>
__global__ void __launch_bounds__(256, 2) conv_brick_kernel(ConvArgs a, const uint16_t *g, float *dx) {
    using B = Brick<ZB, WN>;
    __shared__ __attribute__((aligned(16))) uint16_t Hs[B::NHALO * LDK];
    __shared__ __attribute__((aligned(16))) uint16_t Ws[BR_TG * B::BN * LDK];
    const int tid = threadIdx.x, wv = tid >> 6, l = tid & 63;
    const int cin = DG ? a.cout : a.c1 + a.c2;  // channels summed over (k)
    const int ncol = DG ? a.c1 + a.c2 : a.cout;  // columns of the result
    const int nbx = a.W / BRX, nby = a.H / BRY;
    const int b = blockIdx.x;
    const int x0 = (b % nbx) * BRX, y0 = ((b / nbx) % nby) * BRY, z0 = (b / (nbx * nby)) * ZB;
    const int wm = (wv / WN) * 64, wn = (wv % WN) * 32;
    v16f acc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = 0.0f;
    // halo rows read by this lane's two A blocks (tap offset added per tap)
    int hrow[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int m = wm + 32 * i + (l & 31);
        hrow[i] = ((m >> 6) * HLY + ((m >> 3) & 7)) * HLX + (m & 7);
    }
    // Staging: each thread issues all of a stage's loads into registers and
    // stores them after the barrier that ends the previous stage; the next
    // stage's loads are issued before this stage's MFMAs.
    uint4 hv[B::HL], wr[B::WL];
    brick_fetch_halo<ZB, WN, DG>(a, g, tid, x0, y0, z0, 0, hv);
    brick_fetch_w<ZB, WN, DG>(a, tid, 0, 0, wr);
    for (int c0 = 0; c0 < cin; c0 += BK) {
#pragma unroll
        for (int j = 0; j < B::HL; ++j) {
            const int e = tid + 256 * j;
            if (e < B::NHALO * 4) *reinterpret_cast<uint4 *>(&Hs[(e >> 2) * LDK + 8 * (e & 3)]) = hv[j];
        }
        const int kn = min(BK, cin - c0);
        for (int t0 = 0; t0 < 27; t0 += BR_TG) {
#pragma unroll
            for (int j = 0; j < B::WL; ++j) {
                const int e = tid + 256 * j;
                if (e < B::WE) *reinterpret_cast<uint4 *>(&Ws[(e >> 2) * LDK + 8 * (e & 3)]) = wr[j];
            }
            __syncthreads();
            if (t0 + BR_TG < 27) {
                brick_fetch_w<ZB, WN, DG>(a, tid, c0, t0 + BR_TG, wr);
            } else if (c0 + BK < cin) {
                brick_fetch_halo<ZB, WN, DG>(a, g, tid, x0, y0, z0, c0 + BK, hv);
                brick_fetch_w<ZB, WN, DG>(a, tid, c0 + BK, 0, wr);
            }
            // the stage's nine taps share dz = t0 / 9; unrolled so that the
            // LDS reads of the next taps go out ahead of the MFMAs.  The input
            // gradient reads the halo at the mirrored offset -o_t.
            const int zoff = (DG ? 2 - t0 / BR_TG : t0 / BR_TG) * HLY * HLX;
#pragma unroll
            for (int tt = 0; tt < BR_TG; ++tt) {
                const int toff = DG ? zoff + (2 - tt / 3) * HLX + (2 - tt % 3) : zoff + (tt / 3) * HLX + tt % 3;
#pragma unroll
                for (int kq = 0; kq < 2; ++kq) {
                    if (16 * kq < kn) {  // uniform: the chunk's last channels may end at 8 or 24
                        const int ko = 16 * kq + 8 * (l >> 5);
                        const v8bf fb =
                            *reinterpret_cast<const v8bf *>(&Ws[(tt * B::BN + wn + (l & 31)) * LDK + ko]);
                        const v8bf fa0 = *reinterpret_cast<const v8bf *>(&Hs[(hrow[0] + toff) * LDK + ko]);
                        const v8bf fa1 = *reinterpret_cast<const v8bf *>(&Hs[(hrow[1] + toff) * LDK + ko]);
                        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa0, fb, acc[0], 0, 0, 0);
                        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa1, fb, acc[1], 0, 0, 0);
                    }
                }
            }
            __syncthreads();  // the next stage overwrites the weights (and the halo)
        }
    }
    // D element e of lane l: row 8 (e / 4) + 4 (l / 32) + e % 4, column l % 32
    const int col = wn + (l & 31);
    if (col >= ncol) return;
    const float bias = (!DG && a.b) ? a.b[col] : 0.0f;
    const auto at = [&](int i, int e) {
        const int m = wm + 32 * i + 8 * (e >> 2) + 4 * (l >> 5) + (e & 3);
        return (int64_t(z0 + (m >> 6)) * a.H + (y0 + ((m >> 3) & 7))) * a.W + (x0 + (m & 7));
    };
    if constexpr (DG) {
        if (!a.mg) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) dx[at(i, e) * ncol + col] = acc[i][e];
            return;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            int64_t q[16];
            float v[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                q[e] = at(i, e) * ncol + col;
                v[e] = acc[i][e];
            }
            put_grads(a, dx, q, v);
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int64_t p = at(i, e);
            float v = acc[i][e] + bias;
            if (a.relu) v = fmaxf(v, 0.0f);
            if (a.y) a.y[p * a.cout + col] = f2bf(v);
            if (a.yf) a.yf[p * a.cout + col] = v;
        }
}

// Layers of few positions (the coarse levels).  A work-group of eight
// wavefronts computes a brick of 2 x 4 x 4 positions x 16 NT columns, each
// wavefront parts of K (steps of a tap and 32 channels) for the whole tile.
// The brick's input halo is staged in LDS, SCH channels at a time; the weights'
// operands (16 columns x 32 consecutive channels of one tap) are loaded straight
// from memory into the MFMA registers, the next step's in flight; the
// wavefronts' sums meet in LDS in a fixed order, so no second pass and no
// atomics.  Bound by the weights' way through L1 (one line per column and step).
// 4 096 positions, 128 -> 128 channels: 19 us (191 TFLOP/s); 512: 10.4 us.
// In a network's layers each part is a sum of its own and the parts are added in
// the order of equally fast work-groups, shorter first, last first; otherwise the
// wavefronts' sums run on (17 us against 19 at 4 096 positions, 128 -> 128).
typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int SBZ = 2, SBY = 4, SBX = 4, SHY = SBY + 2, SHX = SBX + 2, SNH = (SBZ + 2) * SHY * SHX;

// gz > 0: K (at most SCH channels, whole operands) in gz parts, each summed from
// zero by a wavefront, and the parts added eight at a time: shorter ones first
// (balanced rounds), the last first among equals; else step s to wavefront s % 8
// and the wavefronts' sums added
template <int NT, bool DG, int SCH>
__global__ void __launch_bounds__(512, 4) conv_small_kernel(ConvArgs a, const uint16_t *g, float *dx, int gz) {
    constexpr int SLD = SCH + 8;  // channels per stage, halo row length
    constexpr int HLB = SNH * SLD * 2, RDB = 8 * 512 * NT * 4;
    __shared__ __attribute__((aligned(16))) char lds[HLB + RDB];
    uint16_t *Hs = reinterpret_cast<uint16_t *>(lds);
    float *sum = reinterpret_cast<float *>(lds + HLB);  // [wavefront][row][column]
    __shared__ int order[27 * SCH / 256 + 1];           // the parts as they are added
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const int cin = a.c1 + a.c2, N = DG ? cin : a.cout, kc = DG ? a.cout : cin;
    const int nbx = (a.W + SBX - 1) / SBX, nby = (a.H + SBY - 1) / SBY, b = blockIdx.x;
    const int x0 = (b % nbx) * SBX, y0 = b / nbx % nby * SBY, z0 = b / (nbx * nby) * SBZ, n0 = blockIdx.y * 16 * NT;
    // operand rows of this lane: position l % 16 of each plane (halo row, the
    // tap's offset is added), column l % 16; its channels 8 (l / 16) .. + 7
    const int k8 = 8 * (l >> 4), hrow = ((l >> 2) & 3) * SHX + (l & 3);
    const uint16_t *wb[NT];
#pragma unroll
    for (int q = 0; q < NT; ++q) {
        const int n = min(n0 + 16 * q + (l & 15), N - 1);
        wb[q] = DG ? a.w + int64_t(n) * a.cout : a.wt + int64_t(n) * 27 * cin;
    }
    const int tstride = DG ? cin * a.cout : cin;  // elements between a column's taps
    const int nall = 27 * ((min(SCH, kc) + 31) / 32);  // steps of the first stage
    if (tid < gz) {
        const auto len = [&](int z) { return nall * (z + 1) / gz - nall * z / gz; };
        int rank = 0;
        for (int z = 0; z < gz; ++z) rank += len(z) < len(tid) || (len(z) == len(tid) && z > tid);
        order[rank] = tid;
    }
    v4f acc[2][NT];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int q = 0; q < NT; ++q) acc[i][q] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    float v[NT];  // elements tid + 512 j of the tile
#pragma unroll
    for (int j = 0; j < NT; ++j) v[j] = 0.0f;
    // adds the sums of the first n wavefronts to v; leaves acc zero
    const auto collect = [&](int n) {
        // D element e of lane l: row 4 (l / 16) + e, column l % 16
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < NT; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sum[wv * 512 * NT + (16 * i + 4 * (l >> 4) + e) * 16 * NT + 16 * q + (l & 15)] = acc[i][q][e];
                    acc[i][q][e] = 0.0f;
                }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int w = 0; w < 8; ++w)
                if (w < n) v[j] += sum[w * 512 * NT + tid + 512 * j];
        __syncthreads();  // read before the next round's stores
    };

    for (int c0 = 0; c0 < kc; c0 += SCH) {
        const int cw = min(SCH, kc - c0), ncc = (cw + 31) / 32, nst = 27 * ncc;
        __syncthreads();  // the previous stage's reads are done
        // halo of channels c0 .. c0 + 127; outside the volume and past the channels: zero
        constexpr int HL = (SNH * (SCH / 8) + 511) / 512;
        uint4 hv[HL];
        bool ok[HL];
#pragma unroll
        for (int j = 0; j < HL; ++j) {
            const int e = tid + 512 * j, hp = min(e / (SCH / 8), SNH - 1), c = c0 + 8 * (e % (SCH / 8));
            const int z = z0 + hp / (SHY * SHX) - 1, y = y0 + hp / SHX % SHY - 1, x = x0 + hp % SHX - 1;
            const int zc = min(max(z, 0), a.D - 1), yc = min(max(y, 0), a.H - 1), xc = min(max(x, 0), a.W - 1);
            ok[j] = c < kc && z == zc && y == yc && x == xc;
            const int cc = min(c, kc - 8);
            const uint16_t *src;
            if constexpr (DG) {
                src = g + ((zc * a.H + yc) * a.W + xc) * a.cout + cc;
            } else {
                const bool skip = cc >= a.c1;
                const int u = !skip && a.up1 ? 1 : 0;
                src = (skip ? a.x2 + cc - a.c1 : a.x1 + cc) +
                      (((zc >> u) * (a.H >> u) + (yc >> u)) * (a.W >> u) + (xc >> u)) * (skip ? a.c2 : a.c1);
            }
            hv[j] = *reinterpret_cast<const uint4 *>(src);
        }
        // the first step's weights
        int z = wv, st = wv, end = 0;
        const auto part = [&]() {  // the z-th to be added: steps st .. end - 1
            const int q = __builtin_amdgcn_readfirstlane(order[min(z, gz - 1)]);
            st = nst * q / gz;
            end = nst * (q + 1) / gz;
        };
        if (gz) part();
        int t = st / ncc, cc = st % ncc;
        bool more = gz ? z < gz : st < nst;  // steps are left for this wavefront
        uint4 wn[NT];
        auto fetch = [&]() {
            // past the channels the last eight of them (read in bounds, then zeroed)
            const int64_t off = int64_t(t) * tstride + c0 + min(32 * cc + k8, cw - 8);
#pragma unroll
            for (int q = 0; q < NT; ++q) wn[q] = *reinterpret_cast<const uint4 *>(wb[q] + off);
        };
        if (more) fetch();
#pragma unroll
        for (int j = 0; j < HL; ++j) {
            const int e = tid + 512 * j;
            if (e < SNH * (SCH / 8))
                *reinterpret_cast<uint4 *>(Hs + e / (SCH / 8) * SLD + 8 * (e % (SCH / 8))) = keep4(ok[j], hv[j]);
        }
        __syncthreads();
        for (int r = 0; r < (gz ? gz : 1); r += 8) {
            bool done = !more;
            while (!done) {
                const int tt = DG ? 26 - t : t, off = (tt / 9 * SHY + tt / 3 % 3) * SHX + tt % 3, c = 32 * cc + k8;
                uint4 w[NT];
#pragma unroll
                for (int q = 0; q < NT; ++q) w[q] = keep4(c < cw, wn[q]);
                if (gz) {
                    done = ++st == end;  // a part ends with this step
                    if (done) {
                        z += 8;
                        part();
                        t = st / ncc;
                        cc = st - t * ncc;
                    } else if (++cc == ncc) {
                        cc = 0;
                        ++t;
                    }
                    more = z < gz;
                } else {
                    st += 8;
                    cc += 8;
                    while (cc >= ncc) {
                        cc -= ncc;
                        ++t;
                    }
                    more = st < nst;
                    done = !more;
                }
                if (more) fetch();
                const uint16_t *hp = Hs + (hrow + off) * SLD + c;
                const v8bf fa0 = *reinterpret_cast<const v8bf *>(hp);
                const v8bf fa1 = *reinterpret_cast<const v8bf *>(hp + SHY * SHX * SLD);
#pragma unroll
                for (int q = 0; q < NT; ++q) {
                    const v8bf fb = __builtin_bit_cast(v8bf, w[q]);
                    acc[0][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa0, fb, acc[0][q], 0, 0, 0);
                    acc[1][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa1, fb, acc[1][q], 0, 0, 0);
                }
            }
            if (gz) collect(min(8, gz - r));
        }
    }
    if (!gz) collect(8);
    int at[NT];  // the element of [P][N], -1 outside
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int e = tid + 512 * j, m = e / (16 * NT), col = n0 + e % (16 * NT);
        const int z = z0 + (m >> 4), y = y0 + (m >> 2 & 3), x = x0 + (m & 3);
        at[j] = z < a.D && y < a.H && x < a.W && col < N ? ((z * a.H + y) * a.W + x) * N + col : -1;
    }
    if constexpr (DG) {
        put_grads(a, dx, at, v);
        return;
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        if (at[j] < 0) continue;
        float r = v[j] + (a.b ? a.b[n0 + (tid + 512 * j) % (16 * NT)] : 0.0f);
        if (a.relu) r = fmaxf(r, 0.0f);
        if (a.y) a.y[at[j]] = f2bf(r);
        if (a.yf) a.yf[at[j]] = r;
    }
}

// packed forward weights: wt[o][k] = w[k][o], k = (tap, input channel), of every layer of the list: one
// work-group per 64 x 64 tile, turned in LDS so that both sides go by lines
// (15 layers, 3.6 M weights: 15 launches of a strided gather 68 us, this one
// launch 11.5)
__global__ void __launch_bounds__(256) pack_weights_kernel(PackList ls) {
    __shared__ uint16_t tile[64][66];
    int L = 0;
    while (L + 1 < ls.n && int(blockIdx.x) >= ls.at[L + 1].tile0) ++L;  // uniform
    const PackLayer p = ls.at[L];
    const int to = (p.cout + 63) / 64, t = blockIdx.x - p.tile0, k0 = t / to * 64, o0 = t % to * 64;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int k = k0 + ty + 4 * r, o = o0 + tx;
        if (k < p.K && o < p.cout) tile[ty + 4 * r][tx] = p.w[int64_t(k) * p.cout + o];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int k = k0 + tx, o = o0 + ty + 4 * r;
        if (k < p.K && o < p.cout) p.wt[int64_t(o) * p.K + k] = tile[tx][ty + 4 * r];
    }
}

// Elementwise passes take V = 8 neighbouring channels (or elements) per thread
// where the channel counts allow and every pointer is 16-byte aligned, else one.
template <int V>
__device__ inline void load_f(const float *p, float (&v)[V]) {
    if constexpr (V == 8) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float4 q = reinterpret_cast<const float4 *>(p)[h];
            v[4 * h] = q.x;
            v[4 * h + 1] = q.y;
            v[4 * h + 2] = q.z;
            v[4 * h + 3] = q.w;
        }
    } else {
        v[0] = p[0];
    }
}
template <int V>
__device__ inline void store_f(float *p, const float (&v)[V]) {
    if constexpr (V == 8) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            reinterpret_cast<float4 *>(p)[h] = make_float4(v[4 * h], v[4 * h + 1], v[4 * h + 2], v[4 * h + 3]);
    } else {
        p[0] = v[0];
    }
}
template <int V>
__device__ inline void load_b(const uint16_t *p, float (&v)[V]) {
    if constexpr (V == 8) {
        const uint4 q = *reinterpret_cast<const uint4 *>(p);
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            v[2 * h] = __uint_as_float(w[h] << 16);
            v[2 * h + 1] = __uint_as_float(w[h] & 0xFFFF0000u);
        }
    } else {
        v[0] = bf2f(p[0]);
    }
}
template <int V>
__device__ inline void store_b(uint16_t *p, const float (&v)[V]) {
    if constexpr (V == 8) {
        uint32_t w[4];
#pragma unroll
        for (int h = 0; h < 4; ++h) w[h] = f2bf(v[2 * h]) | uint32_t(f2bf(v[2 * h + 1])) << 16;
        *reinterpret_cast<uint4 *>(p) = make_uint4(w[0], w[1], w[2], w[3]);
    } else {
        p[0] = f2bf(v[0]);
    }
}

// g = BF16(dy (y > 0)) (or BF16(dy) without the ReLU)
template <int V>
__global__ void relu_grad_kernel(const float *dy, const uint16_t *y, int64_t n, int relu, uint16_t *g) {
    for (int64_t i = (blockIdx.x * int64_t(blockDim.x) + threadIdx.x) * V; i < n; i += int64_t(gridDim.x) * blockDim.x * V) {
        float v[V], m[V];
        load_f<V>(dy + i, v);
        if (relu) {
            load_b<V>(y + i, m);
#pragma unroll
            for (int q = 0; q < V; ++q) v[q] = m[q] > 0.0f ? v[q] : 0.0f;
        }
        store_b<V>(g + i, v);
    }
}

// Weight gradient dw[t, c, o] += sum_p x[p + o_t, c] g[p, o]: a work-group owns
// 32 input channels, 32 output channels, the nine taps of one dz and a share of
// the volume's bricks of 4 x 8 x 8 positions; each wavefront takes one plane of
// a brick and keeps the nine taps' 32 x 32 sums in registers.  Per brick the
// input halo of the four shifted planes and g are staged in LDS once, position
// by position as they lie in memory; the MFMA operands need eight positions of
// one channel per lane, which the transposing LDS read delivers
// (ds_read_b64_tr_b16: lane i of 16 gets element i % 4 of lanes i / 4 + 4 q,
// q = 0..3, so four positions of its channel).
//
// Bound by the LDS reads (one KB per tap and 16 positions against one MFMA)
// and by the FP32 atomics into dw: 200 G/s with every work-group adding to the
// same addresses, which is why a work-group holds nine taps and not all 27
// (three times the sums for the same number of work-groups). The 15
// layers of the 128 x 64 x 32 canvas take 0.41 ms (0.34 without the atomics)
// against 1.02 ms for a GEMM over (tap, channel) rows that staged x again for
// each row tile, transposed it with 2-byte LDS writes and summed the bias in a
// pass of its own; the 64 + 32 -> 32 layer 65 us (660 TFLOP/s) against 194.
//
typedef short v4s __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v8bf read_tr(const char *p, int step) {
    typedef __attribute__((address_space(3))) v4s lds_v4s;
    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s *)(p));
    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s *)(p + step));
    return __builtin_bit_cast(v8bf, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

__global__ void __launch_bounds__(256, 2) conv_wgrad_kernel(ConvArgs a, const uint16_t *g, float *dw, float *db) {
    constexpr int PS = LDK * 2;  // bytes per position in LDS
    constexpr int NX = 4 * HLY * HLX, XL = (NX * 4 + 255) / 256, GL = 4;
    __shared__ __attribute__((aligned(16))) char Xs[(NX + 256) * PS];
    char *Gs = Xs + NX * PS;
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const int cin = a.c1 + a.c2, c0 = int(blockIdx.y / 3) * 32, dz = int(blockIdx.y % 3) - 1, o0 = blockIdx.z * 32;
    const int nbx = (a.W + BRX - 1) / BRX, nby = (a.H + BRY - 1) / BRY, nb = nbx * nby * ((a.D + 3) / 4);
    // this lane's operand address: position row (l % 16) / 4 of its k-group's
    // four, channels 16 (l / 16 % 2) + 4 (l % 4) .. + 3; k-group l / 32 is the
    // brick row below
    const int kr = (l >> 2) & 3, kg = l >> 5, cb = ((l >> 4) & 1) * 32 + (l & 3) * 8;
    const char *xl = Xs + ((wv * HLY + kg) * HLX + kr) * PS + cb;
    const char *gl = Gs + ((wv * BRY + kg) * BRX + kr) * PS + cb;
    v16f acc[9];
#pragma unroll
    for (int j = 0; j < 9; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][e] = 0.0f;
    float bsum[8] = {0, 0, 0, 0, 0, 0, 0, 0};  // g over this thread's positions, channels 8 (tid % 4) ..
    const bool bias = db && blockIdx.y == 0;

    // a thread loads the same eight channels of x and of g everywhere; a
    // position outside the volume reads the nearest one inside and becomes zero
    const int cx8 = c0 + 8 * (tid & 3), co8 = o0 + 8 * (tid & 3);
    const bool skip = cx8 >= a.c1;
    const int up = !skip && a.up1 ? 1 : 0, cs = skip ? a.c2 : a.c1;
    const bool con = cx8 < cin, oon = co8 < a.cout;
    const uint16_t *xs = con ? (skip ? a.x2 + cx8 - a.c1 : a.x1 + cx8) : a.x1, *gs = oon ? g + co8 : g;
    const int Hs = a.H >> up, Ws = a.W >> up, css = con ? cs : 0, cgs = oon ? a.cout : 0;
    uint4 hv[XL], gv[GL];
    unsigned inside = 0;  // bit per load
    auto fetch = [&](int b) {
        const int x0 = (b % nbx) * BRX, y0 = (b / nbx % nby) * BRY, z0 = (b / (nbx * nby)) * 4;
        bool ok[XL + GL];
#pragma unroll
        for (int j = 0; j < XL; ++j) {
            const int hp = min((tid >> 2) + 64 * j, NX - 1);
            const int z = z0 + hp / (HLY * HLX) + dz, y = y0 + hp / HLX % HLY - 1, x = x0 + hp % HLX - 1;
            const int zc = min(max(z, 0), a.D - 1), yc = min(max(y, 0), a.H - 1), xc = min(max(x, 0), a.W - 1);
            ok[j] = con && z == zc && y == yc && x == xc;
            hv[j] = *reinterpret_cast<const uint4 *>(xs + (((zc >> up) * Hs + (yc >> up)) * Ws + (xc >> up)) * css);
        }
#pragma unroll
        for (int j = 0; j < GL; ++j) {
            const int z = z0 + j, y = y0 + (tid >> 5), x = x0 + (tid >> 2 & 7);
            const int zc = min(z, a.D - 1), yc = min(y, a.H - 1), xc = min(x, a.W - 1);
            ok[XL + j] = oon && z == zc && y == yc && x == xc;
            gv[j] = *reinterpret_cast<const uint4 *>(gs + ((zc * a.H + yc) * a.W + xc) * cgs);
        }
        inside = 0;
#pragma unroll
        for (int j = 0; j < XL + GL; ++j) inside |= ok[j] ? 1u << j : 0u;
    };
    // this work-group's bricks: a contiguous range
    const int nw = gridDim.x, b0 = int(int64_t(nb) * blockIdx.x / nw), b1 = int(int64_t(nb) * (blockIdx.x + 1) / nw);
    fetch(b0);
    for (int b = b0; b < b1; ++b) {
        __syncthreads();  // the previous brick's reads are done
#pragma unroll
        for (int j = 0; j < XL; ++j) {
            const int e = tid + 256 * j;
            if (e < NX * 4)
                *reinterpret_cast<uint4 *>(Xs + (e >> 2) * PS + 16 * (e & 3)) = keep4(inside >> j & 1u, hv[j]);
        }
#pragma unroll
        for (int j = 0; j < GL; ++j) {
            gv[j] = keep4(inside >> (XL + j) & 1u, gv[j]);
            *reinterpret_cast<uint4 *>(Gs + ((tid >> 2) + 64 * j) * PS + 16 * (tid & 3)) = gv[j];
            if (bias) {
                const uint32_t w[4] = {gv[j].x, gv[j].y, gv[j].z, gv[j].w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    bsum[2 * q] += __uint_as_float(w[q] << 16);
                    bsum[2 * q + 1] += __uint_as_float(w[q] & 0xFFFF0000u);
                }
            }
        }
        __syncthreads();
        if (b + 1 < b1) fetch(b + 1);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {  // 16 positions: two rows of the wavefront's plane
            const v8bf fb = read_tr(gl + ks * 16 * PS, 4 * PS);
#pragma unroll
            for (int j = 0; j < 9; ++j) {
                const v8bf fa = read_tr(xl + ((2 * ks + j / 3) * HLX + j % 3) * PS, 4 * PS);
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb, acc[j], 0, 0, 0);
            }
        }
    }
    // the four wavefronts' sums meet in LDS, three taps at a time ([wavefront]
    // [tap][channel][32]), and go out (LDS float atomics instead took 40 us);
    // D element e of lane l: row (channel) 8 (e / 4) + 4 (l / 32) + e % 4, column l % 32
    float *sum = reinterpret_cast<float *>(Xs);
    float *own = sum + wv * 3072 + 4 * (l >> 5) * 32 + (l & 31);
#pragma unroll
    for (int j0 = 0; j0 < 9; j0 += 3) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) own[(j * 32 + 8 * (e >> 2) + (e & 3)) * 32] = acc[j0 + j][e];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 12; ++q) {
            const int e = tid + 256 * q, row = e >> 5 & 31, col = e & 31;
            const float v = (sum[e] + sum[3072 + e]) + (sum[6144 + e] + sum[9216 + e]);
            if (c0 + row < cin && o0 + col < a.cout)
                atomicAdd(dw + (int64_t(9 * (dz + 1) + j0 + (e >> 10)) * cin + c0 + row) * a.cout + o0 + col, v);
        }
    }
    if (bias) {  // uniform; one atomic instruction per work-group: all add to the same line
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 8; ++q) {
#pragma unroll
            for (int o = 4; o < 64; o <<= 1) bsum[q] += __shfl_xor(bsum[q], o, 64);
            if (l < 4) sum[32 * wv + 8 * l + q] = bsum[q];
        }
        __syncthreads();
        if (tid < 32 && o0 + tid < a.cout)
            atomicAdd(db + o0 + tid, (sum[tid] + sum[32 + tid]) + (sum[64 + tid] + sum[96 + tid]));
    }
}

// ---------------------------------------------------------------------------
// pooling and the gradient plumbing of the U-Net
// ---------------------------------------------------------------------------
// a volume's extents for the passes below: element e = (position, channel group)
struct Vol {
    int D, H, W, C;  // the coarser volume, channels
    int64_t n;       // elements
    int w, h;        // extents of the volume that is run over
    Divider by_c, by_w, by_h;
    // coordinates of element e (the dividers hold up to 2^31 of them)
    template <int V>
    __device__ void at(int64_t e, int64_t &q, int &x, int &y, int &z, int &c) const {
        if (n < (int64_t(1) << 31)) {
            const uint32_t q32 = by_c(uint32_t(e)), r = by_w(q32);
            q = q32;
            z = by_h(r);
            x = q32 - r * w;
            y = r - uint32_t(z) * h;
        } else {
            q = e / (C / V);
            x = int(q % w);
            y = int(q / w % h);
            z = int(q / w / h);
        }
        c = V * int(e - q * (C / V));
    }
};
// y[q, c] = mean of the 8 children of q (BF16 in, BF16 out)
template <int V>
__global__ void pool2_kernel(const uint16_t *x, Vol vol, uint16_t *y) {
    const int W = 2 * vol.W, H = 2 * vol.H;
    for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < vol.n; e += int64_t(gridDim.x) * blockDim.x) {
        int64_t q;
        int qw, qh, qd, c;
        vol.at<V>(e, q, qw, qh, qd, c);
        float s[V], v[8][V];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int64_t p = (int64_t(2 * qd + (j >> 2)) * H + 2 * qh + ((j >> 1) & 1)) * W + 2 * qw + (j & 1);
            load_b<V>(x + p * vol.C + c, v[j]);
        }
#pragma unroll
        for (int u = 0; u < V; ++u) {
            s[u] = 0.0f;
#pragma unroll
            for (int j = 0; j < 8; ++j) s[u] += v[j][u];
            s[u] *= 0.125f;
        }
        store_b<V>(y + e * V, s);
    }
}

// g[p, c] = gc[parent(p), c] / 8 (+ skip[p, off + c] when skip is given); with my,
// BF16(g (my > 0)) into gb instead (the gradient of the ReLU layer below)
template <int V>
__global__ void pool2_back_kernel(const float *gc, const float *skip, int skip_stride, int skip_off, Vol vol,
                                  const uint16_t *my, float *g, uint16_t *gb) {
    for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < vol.n; e += int64_t(gridDim.x) * blockDim.x) {
        int64_t p;
        int pw, ph, pd, c;
        vol.at<V>(e, p, pw, ph, pd, c);
        const int64_t q = (int64_t(pd >> 1) * vol.H + (ph >> 1)) * vol.W + (pw >> 1);
        float v[V], k[V], m[V];
        load_f<V>(gc + q * vol.C + c, v);
        if (skip) load_f<V>(skip + p * skip_stride + skip_off + c, k);
        if (my) load_b<V>(my + e * V, m);
#pragma unroll
        for (int u = 0; u < V; ++u) {
            v[u] *= 0.125f;
            if (skip) v[u] += k[u];
            if (my) v[u] = m[u] > 0.0f ? v[u] : 0.0f;
        }
        if (my) store_b<V>(gb + e * V, v);
        else store_f<V>(g + e * V, v);
    }
}

// gc[q, c] = sum over the 8 children p of q of g[p, c] (g row stride `stride`);
// with my, BF16(gc (my > 0)) into gb instead
template <int V>
__global__ void up2_back_kernel(const float *g, int stride, Vol vol, const uint16_t *my, float *gc, uint16_t *gb) {
    const int W = 2 * vol.W, H = 2 * vol.H;
    for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < vol.n; e += int64_t(gridDim.x) * blockDim.x) {
        int64_t q;
        int qw, qh, qd, c;
        vol.at<V>(e, q, qw, qh, qd, c);
        float s[V], v[8][V], m[V];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int64_t p = (int64_t(2 * qd + (j >> 2)) * H + 2 * qh + ((j >> 1) & 1)) * W + 2 * qw + (j & 1);
            load_f<V>(g + p * stride + c, v[j]);
        }
        if (my) load_b<V>(my + e * V, m);
#pragma unroll
        for (int u = 0; u < V; ++u) {
            s[u] = 0.0f;
#pragma unroll
            for (int j = 0; j < 8; ++j) s[u] += v[j][u];
            if (my) s[u] = m[u] > 0.0f ? s[u] : 0.0f;
        }
        if (my) store_b<V>(gb + e * V, s);
        else store_f<V>(gc + e * V, s);
    }
}

__global__ void fill_f32_kernel(float *p, int64_t n, float v) {
    for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x) p[i] = v;
}

// ---------------------------------------------------------------------------
// loss in channel-normalised units: pred = xin[:, 0:6] + s * out[:, 0:6],
// e_c = (pred_c - tgt_c) / s_c, loss = masked mean of e^2 over the six
// channels + lam (relative rho_A mass error)^2; tensors [P][8] FP32, mask =
// xin[:, 6]
// ---------------------------------------------------------------------------
constexpr int LOSS_BLOCKS = 256;

__global__ void __launch_bounds__(256) loss_partial_kernel(const float *out, const float *xin, const float *tgt, int64_t P,
                                                           ChanScale sc, double *part) {
    __shared__ double sh[4][4];
    double s[4] = {0, 0, 0, 0};  // sum mask, sum mask tgt_A, sum mask (pred_A - tgt_A), sum mask e^2
    for (int64_t p = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; p < P; p += int64_t(gridDim.x) * blockDim.x) {
        const float m = xin[p * 8 + 6];
        if (m == 0.0f) continue;
        double sq = 0.0;
        for (int c = 0; c < 6; ++c) {
            const double d = (double(xin[p * 8 + c]) + double(sc.s[c]) * double(out[p * 8 + c]) - double(tgt[p * 8 + c])) /
                             double(sc.s[c]);
            sq += d * d;
        }
        s[0] += m;
        s[1] += m * double(tgt[p * 8]);
        s[2] += m * (double(xin[p * 8]) + double(sc.s[0]) * double(out[p * 8]) - double(tgt[p * 8]));
        s[3] += m * sq;
    }
    for (int q = 0; q < 4; ++q) {
        double v = s[q];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6][q] = v;
    }
    __syncthreads();
    if (threadIdx.x < 4) part[blockIdx.x * 4 + threadIdx.x] = sh[0][threadIdx.x] + sh[1][threadIdx.x] +
                                                            sh[2][threadIdx.x] + sh[3][threadIdx.x];
}

// totals in a fixed order (one wavefront: strided over its lanes, then a
// butterfly; one thread took 26 us); res = sum mask, sum mask tgt_A, mass error, loss
__global__ void __launch_bounds__(64) loss_total_kernel(const double *part, int nb, double lam, double *res) {
    double s[4] = {0, 0, 0, 0};
    for (int b = threadIdx.x; b < nb; b += 64)
        for (int q = 0; q < 4; ++q) s[q] += part[b * 4 + q];
    for (int q = 0; q < 4; ++q)
        for (int o = 32; o > 0; o >>= 1) s[q] += __shfl_xor(s[q], o, 64);
    if (threadIdx.x != 0) return;
    const double me = s[1] != 0.0 ? s[2] / s[1] : 0.0;
    res[0] = s[0];
    res[1] = s[1];
    res[2] = me;
    res[3] = (s[0] > 0.0 ? s[3] / (6.0 * s[0]) : 0.0) + lam * me * me;
}

__global__ void loss_grad_kernel(const float *out, const float *xin, const float *tgt, int64_t P, ChanScale sc,
                                 double lam, const double *res, float *grad) {
    const double n = res[0], mt = res[1], me = res[2];
    for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < P * 8; e += int64_t(gridDim.x) * blockDim.x) {
        const int64_t p = e >> 3;
        const int c = int(e & 7);
        const float m = xin[p * 8 + 6];
        double g = 0.0;
        if (c < 6 && m != 0.0f && n > 0.0) {
            const double sc_c = sc.s[c];
            const double d = (double(xin[e]) + sc_c * double(out[e]) - double(tgt[e])) / sc_c;
            g = 2.0 * m * d / (6.0 * n);
            if (c == 0 && mt != 0.0) g += 2.0 * lam * me * m * sc_c / mt;
        }
        grad[e] = float(g);
    }
}

// per-channel sums of mask (y - x)^2 and of the mask over one pair of canvases
__global__ void __launch_bounds__(256) moments_kernel(const float *x, const float *y, int64_t P, double *part) {
    __shared__ double sh[4][7];
    double s[7] = {0, 0, 0, 0, 0, 0, 0};
    for (int64_t p = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; p < P; p += int64_t(gridDim.x) * blockDim.x) {
        const double m = x[p * 8 + 6];
        if (m == 0.0) continue;
        for (int c = 0; c < 6; ++c) {
            const double d = double(y[p * 8 + c]) - double(x[p * 8 + c]);
            s[c] += m * d * d;
        }
        s[6] += m;
    }
    for (int q = 0; q < 7; ++q) {
        double v = s[q];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6][q] = v;
    }
    __syncthreads();
    if (threadIdx.x < 7) part[blockIdx.x * 7 + threadIdx.x] = sh[0][threadIdx.x] + sh[1][threadIdx.x] +
                                                            sh[2][threadIdx.x] + sh[3][threadIdx.x];
}

__global__ void moments_total_kernel(const double *part, int nb, double *res) {
    if (threadIdx.x != 0) return;
    double s[7] = {0, 0, 0, 0, 0, 0, 0};
    for (int b = 0; b < nb; ++b)
        for (int q = 0; q < 7; ++q) s[q] += part[b * 7 + q];
    for (int q = 0; q < 7; ++q) res[q] = s[q];
}

// ---------------------------------------------------------------------------
// Adam on FP32 master parameters, with the BF16 copy the kernels read
// ---------------------------------------------------------------------------
__global__ void adam_kernel(float *p, const float *g, float *m, float *v, uint16_t *pb, int64_t n, float lr, float b1,
                            float b2, float eps, float c1, float c2) {
    for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.0f - b1) * gi;
        const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
        p[i] = pi;
        if (pb) pb[i] = f2bf(pi);
    }
}

// prediction of the network: pred[:, 0:6] = xin[:, 0:6] + s * out[:, 0:6], the rest
// copied from the input; also the BF16 copy (next input of a rollout)
__global__ void residual_kernel(const float *out, const float *xin, int64_t P, ChanScale sc, float *pred,
                                uint16_t *predb) {
    for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < P * 8; e += int64_t(gridDim.x) * blockDim.x) {
        const int c = int(e & 7);
        const float v = c < 6 ? xin[e] + sc.s[c] * out[e] : xin[e];
        if (pred) pred[e] = v;
        if (predb) predb[e] = f2bf(v);
    }
}

// network input: y[:, c] = BF16((x[:, c] - shift[c]) * gain[c]) on [P][8] cells
__global__ void normalize_kernel(const float *x, int64_t P, ChanScale shift, ChanScale gain, uint16_t *y) {
    for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < P * 8; e += int64_t(gridDim.x) * blockDim.x) {
        const int c = int(e & 7);
        y[e] = f2bf((x[e] - shift.s[c]) * gain.s[c]);
    }
}

__global__ void to_bf16_kernel(const float *x, int64_t n, uint16_t *y) {
    for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
        y[i] = f2bf(x[i]);
}

// ---------------------------------------------------------------------------
// restriction and lift
//
// Both work with the physical velocity u = (j + F/2) / rho of the method
// (Shan-Chen force F of the fused step, velocity shift of the collision).  The stored state is the
// collision output f*, whose momentum is j* = j + F for equal relaxation
// times, so a restriction reads u = (j* - F/2) / rho with F from the stored
// densities, and a lift writes f*_k = f^eq(rho_k, u - F/(2 rho) + tau_k F_k /
// rho_k) with F from the lifted densities.  The force needs psi of the
// neighbours: a first pass writes psi_k of every node to scratch.
// ---------------------------------------------------------------------------
__device__ inline double psi_solid(const SurLattice &L, uint8_t m, int k) {
    return L.psi_tab[2 * (m & MAT_ID_MASK) + k];
}

// F_k = -G psi_k(x) sum_i w_i psi_kbar(x + c_i) c_i + rho_k g at fluid node
// (x, y, z) with densities rho (= psi on fluid).  A fluid node never reaches
// beyond a closed end plane (the end planes are solid), so the neighbours'
// coordinates are wrapped or clamped without a test and all loads are
// issued together.
__device__ inline void force_at(const SurLattice &L, int x, int y, int z, const double rho[2], double F[2][3]) {
    const int64_t n_all = int64_t(L.nx) * L.ny * L.nz;
    const int xs[3] = {x > 0 ? x - 1 : (L.px ? L.nx - 1 : 0), x, x + 1 < L.nx ? x + 1 : (L.px ? 0 : x)};
    const int ys[3] = {y > 0 ? y - 1 : (L.py ? L.ny - 1 : 0), y, y + 1 < L.ny ? y + 1 : (L.py ? 0 : y)};
    const int zs[3] = {z > 0 ? z - 1 : (L.pz ? L.nz - 1 : 0), z, z + 1 < L.nz ? z + 1 : (L.pz ? 0 : z)};
    double p[2][Q];
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        const int64_t m = (int64_t(zs[1 + cz(i)]) * L.ny + ys[1 + cy(i)]) * L.nx + xs[1 + cx(i)];
        p[0][i] = gptr(L.psi)[m];
        p[1][i] = gptr(L.psi)[n_all + m];
    }
    double s[2][3] = {{0, 0, 0}, {0, 0, 0}};
#pragma unroll
    for (int i = 1; i < Q; ++i)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const double v = wgt<double>(i) * p[1 - k][i];
            if (cx(i)) s[k][0] += v * cx(i);
            if (cy(i)) s[k][1] += v * cy(i);
            if (cz(i)) s[k][2] += v * cz(i);
        }
    for (int k = 0; k < 2; ++k)
        for (int d = 0; d < 3; ++d) F[k][d] = -L.G * rho[k] * s[k][d] + rho[k] * L.g[d];
}

// psi_k of the stored state (rho_k on fluid nodes, the material's value
// elsewhere) and the fluid nodes' momentum sum_k j*_k into rows 2..4 of the
// same scratch, so that the populations are read once: the cells then read
// 40 bytes a node instead of every population again (256 x 128 x 64 FP32, both
// passes: 232 -> 150 us)
template <class S>
__global__ void psi_state_kernel(const S *f, SurLattice L) {
    const int64_t n_all = int64_t(L.nx) * L.ny * L.nz;
    for (int64_t n = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; n < n_all; n += int64_t(gridDim.x) * blockDim.x) {
        const uint8_t m = L.mat[n];
        if ((m & MAT_ID_MASK) != MAT_FLUID) {
            for (int k = 0; k < 2; ++k) L.psi[k * n_all + n] = psi_solid(L, m, k);
            continue;
        }
        double j[3] = {0, 0, 0};
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            double r = 0.0;
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                const double v = double(Codec<S>::dec(f[(k * Q + i) * L.fs + n])) + wgt<double>(i) * L.rref[k];
                r += v;
                if (cx(i)) j[0] += v * cx(i);
                if (cy(i)) j[1] += v * cy(i);
                if (cz(i)) j[2] += v * cz(i);
            }
            L.psi[k * n_all + n] = r;
        }
        for (int d = 0; d < 3; ++d) L.psi[(2 + d) * n_all + n] = j[d];
    }
}

// Eight lanes per cell, one per node of its 2 x 2 x 2 block; the block sums by
// xor butterflies, and lane q writes channel q: 82 us on the 128 x 64 x 32
// canvas (125 us while the force waited for each neighbour behind its bounds
// test).
__global__ void __launch_bounds__(256) restrict_kernel(SurLattice L, int D, int H, int W, float *outf, uint16_t *outb) {
    const int64_t P = int64_t(D) * H * W, n_all = int64_t(L.nx) * L.ny * L.nz;
    const int nx = L.nx, ny = L.ny, nz = L.nz, q = threadIdx.x & 7;
    // each XCD takes a contiguous range of cells: the force's stencil re-reads
    // psi of neighbouring rows and planes, which then stay in one L2
    const int g = gridDim.x, b = (g & 7) == 0 ? int(blockIdx.x & 7) * (g >> 3) + int(blockIdx.x >> 3) : int(blockIdx.x);
    for (int64_t c0 = b * int64_t(32); c0 < P; c0 += int64_t(g) * 32) {
        const int64_t c = c0 + (threadIdx.x >> 3);
        const int64_t row = P >> 32 ? c / W : int64_t(uint32_t(c) / uint32_t(W));
        const int qx = int(c - row * W);
        const int qz = P >> 32 ? int(row / H) : int(uint32_t(row) / uint32_t(H)), qy = int(row - int64_t(qz) * H);
        const bool in = c < P && 2 * qz + 1 < nz && 2 * qy + 1 < ny && 2 * qx + 1 < nx;
        double v[5] = {0, 0, 0, 0, 0};  // rho_A, rho_B, momentum of the node
        int nf = 0, nrod = 0;
        if (in) {
            const int z = 2 * qz + (q >> 2), y = 2 * qy + ((q >> 1) & 1), x = 2 * qx + (q & 1);
            const int64_t n = (int64_t(z) * ny + y) * nx + x;
            const uint8_t m = L.mat[n] & MAT_ID_MASK;
            nrod = m == MAT_ROD;
            nf = m == MAT_FLUID;
            if (nf) {
                const double r[2] = {L.psi[n], L.psi[n_all + n]};
                double F[2][3];
                force_at(L, x, y, z, r, F);
                v[0] = r[0];
                v[1] = r[1];
                for (int d = 0; d < 3; ++d) v[2 + d] = L.psi[(2 + d) * n_all + n] - 0.5 * (F[0][d] + F[1][d]);
            }
        }
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) {
#pragma unroll
            for (int d = 0; d < 5; ++d) v[d] += __shfl_xor(v[d], o, 64);
            nf += __shfl_xor(nf, o, 64);
            nrod += __shfl_xor(nrod, o, 64);
        }
        if (c >= P) continue;
        float cell;
        if (!in) {
            cell = q == 0 ? 0.03f : (q == 1 ? 1.0f : 0.0f);
        } else {
            const double tot = v[0] + v[1];
            const double dens = q == 0 ? v[0] : v[1], mom = q == 2 ? v[2] : (q == 3 ? v[3] : v[4]);
            cell = q < 2    ? (nf ? float(dens / nf) : 0.0f)
                   : q < 5  ? (nf && tot > 0.0 ? float(mom / tot) : 0.0f)
                   : q == 5 ? float(nrod / 8.0)
                   : q == 6 ? 1.0f
                            : float(nf / 8.0);
        }
        if (outf) outf[c * 8 + q] = cell;
        if (outb) outb[c * 8 + q] = f2bf(cell);
    }
}

__device__ inline void lerp_index(int x, int nc, int &i0, int &i1, double &w) {
    double c = x / 2.0 - 0.25;
    c = fmin(fmax(c, 0.0), nc - 1.0);
    i0 = int(floor(c));
    i1 = min(i0 + 1, nc - 1);
    w = c - i0;
}

// prolonged (rho_A, rho_B, u) at fine node (x, y, z): trilinear over the
// corner cells that hold fluid (channel 7 > 0), renormalised; else the plain
// mean of the fluid-holding cells of the 4 x 4 x 4 block around them; else
// gas at rest
__device__ inline void prolong_at(const float *coarse, int H, int W, int ncz, int ncy, int ncx, int x, int y, int z,
                                  double a[5]) {
    int z0, z1, y0, y1, x0, x1;
    double wz, wy, wx;
    lerp_index(z, ncz, z0, z1, wz);
    lerp_index(y, ncy, y0, y1, wy);
    lerp_index(x, ncx, x0, x1, wx);
    for (int q = 0; q < 5; ++q) a[q] = 0.0;
    double wsum = 0.0;
    for (int j = 0; j < 8; ++j) {
        const int iz = (j >> 2) ? z1 : z0, iy = ((j >> 1) & 1) ? y1 : y0, ix = (j & 1) ? x1 : x0;
        const double fz = (j >> 2) ? wz : 1.0 - wz, fy = ((j >> 1) & 1) ? wy : 1.0 - wy, fx = (j & 1) ? wx : 1.0 - wx;
        const float *cc = coarse + ((int64_t(iz) * H + iy) * W + ix) * 8;
        if (!(cc[7] > 0.0f)) continue;
        const double wt = fz * fy * fx;
        for (int q = 0; q < 5; ++q) a[q] += wt * double(cc[q]);
        wsum += wt;
    }
    if (wsum > 0.0) {
        for (int q = 0; q < 5; ++q) a[q] /= wsum;
        return;
    }
    int cnt = 0;
    for (int iz = z0 - 1; iz <= z0 + 2; ++iz)
        for (int iy = y0 - 1; iy <= y0 + 2; ++iy)
            for (int ix = x0 - 1; ix <= x0 + 2; ++ix) {
                if (iz < 0 || iz >= ncz || iy < 0 || iy >= ncy || ix < 0 || ix >= ncx) continue;
                const float *cc = coarse + ((int64_t(iz) * H + iy) * W + ix) * 8;
                if (!(cc[7] > 0.0f)) continue;
                for (int q = 0; q < 5; ++q) a[q] += double(cc[q]);
                ++cnt;
            }
    if (cnt) {
        for (int q = 0; q < 5; ++q) a[q] /= cnt;
    } else {
        a[0] = 0.03;
        a[1] = 1.0;
    }
}

// Largest lifted speed: half the lattice's |u| > 0.3 stability flag.  A
// predicted canvas can hold negative densities or such speeds, which the
// method's own states never do; the lift maps each prolonged node back: rho_k
// clamped at 0, u scaled down to this speed with its direction kept.
constexpr double kLiftSpeedMax = 0.15;

__device__ inline void make_admissible(double a[5]) {
    a[0] = fmax(a[0], 0.0);
    a[1] = fmax(a[1], 0.0);
    const double sp = sqrt(a[2] * a[2] + a[3] * a[3] + a[4] * a[4]);
    if (sp > kLiftSpeedMax) {
        const double sc = kLiftSpeedMax / sp;
        for (int d = 2; d < 5; ++d) a[d] *= sc;
    }
}

// The lift keeps each component's mass: after the admissible map, rho_k on
// the fluid nodes is scaled by s_k = (canvas total of rho_k x fluid nodes of
// each cell) / (lifted total), when both totals are positive.  First the
// lifted totals, per block in a fixed order (grid-stride nodes per thread,
// then a tree over the block) ...
__global__ void __launch_bounds__(256) lift_mass_kernel(const float *coarse, int H, int W, SurLattice L, double *part) {
    __shared__ double red[2][256];
    const int64_t n_all = int64_t(L.nx) * L.ny * L.nz;
    double t[2] = {0.0, 0.0};
    for (int64_t n = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; n < n_all; n += int64_t(gridDim.x) * blockDim.x) {
        if ((L.mat[n] & MAT_ID_MASK) != MAT_FLUID) continue;
        const int x = int(n % L.nx), y = int((n / L.nx) % L.ny), z = int(n / (int64_t(L.nx) * L.ny));
        double a[5];
        prolong_at(coarse, H, W, L.nz / 2, L.ny / 2, L.nx / 2, x, y, z, a);
        make_admissible(a);
        t[0] += a[0];
        t[1] += a[1];
    }
    red[0][threadIdx.x] = t[0];
    red[1][threadIdx.x] = t[1];
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h) {
            red[0][threadIdx.x] += red[0][threadIdx.x + h];
            red[1][threadIdx.x] += red[1][threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x < 2) part[2 * blockIdx.x + threadIdx.x] = red[threadIdx.x][0];
}

// ... then, in one work-group, the canvas totals over the cells inside the
// lattice, the blocks' totals in block order, and the two factors
__global__ void __launch_bounds__(256) lift_scale_kernel(const float *coarse, int H, int W, SurLattice L,
                                                         const double *part, int nb, double *scale) {
    __shared__ double red[4][256];
    const int ncz = L.nz / 2, ncy = L.ny / 2, ncx = L.nx / 2;
    const int64_t ncell = int64_t(ncz) * ncy * ncx;
    double t[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t c = threadIdx.x; c < ncell; c += blockDim.x) {
        const int cx = int(c % ncx), cy = int((c / ncx) % ncy), cz = int(c / (int64_t(ncx) * ncy));
        const float *cc = coarse + ((int64_t(cz) * H + cy) * W + cx) * 8;
        const double nf = 8.0 * double(cc[7]);
        t[0] += double(cc[0]) * nf;
        t[1] += double(cc[1]) * nf;
    }
    for (int b = threadIdx.x; b < nb; b += blockDim.x) {
        t[2] += part[2 * b];
        t[3] += part[2 * b + 1];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) red[q][threadIdx.x] = t[q];
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h)
#pragma unroll
            for (int q = 0; q < 4; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x < 2) {
        const double want = red[threadIdx.x][0], have = red[2 + threadIdx.x][0];
        scale[threadIdx.x] = (want > 0.0 && have > 0.0) ? want / have : 1.0;
    }
}

// psi_k of the lifted state: prolonged rho_k on fluid nodes, the material's value elsewhere
__global__ void psi_lift_kernel(const float *coarse, int H, int W, SurLattice L, const double *scale) {
    const int64_t n_all = int64_t(L.nx) * L.ny * L.nz;
    for (int64_t n = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; n < n_all; n += int64_t(gridDim.x) * blockDim.x) {
        const uint8_t m = L.mat[n];
        double v[2];
        if ((m & MAT_ID_MASK) == MAT_FLUID) {
            const int x = int(n % L.nx), y = int((n / L.nx) % L.ny), z = int(n / (int64_t(L.nx) * L.ny));
            double a[5];
            prolong_at(coarse, H, W, L.nz / 2, L.ny / 2, L.nx / 2, x, y, z, a);
            make_admissible(a);
            v[0] = a[0] * scale[0];
            v[1] = a[1] * scale[1];
        } else {
            v[0] = psi_solid(L, m, 0);
            v[1] = psi_solid(L, m, 1);
        }
        L.psi[n] = v[0];
        L.psi[n_all + n] = v[1];
    }
}

template <class S>
__global__ void lift_kernel(const float *coarse, int H, int W, SurLattice L, const double *scale, S *f) {
    const int64_t n_all = int64_t(L.nx) * L.ny * L.nz;
    for (int64_t n = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; n < n_all; n += int64_t(gridDim.x) * blockDim.x) {
        if ((L.mat[n] & MAT_ID_MASK) != MAT_FLUID) continue;
        const int x = int(n % L.nx), y = int((n / L.nx) % L.ny), z = int(n / (int64_t(L.nx) * L.ny));
        double a[5];
        prolong_at(coarse, H, W, L.nz / 2, L.ny / 2, L.nx / 2, x, y, z, a);
        make_admissible(a);
        const double rho[2] = {a[0] * scale[0], a[1] * scale[1]};
        double F[2][3];
        force_at(L, x, y, z, rho, F);
        const double tot = rho[0] + rho[1];
        const double ih = tot > 1e-12 ? 0.5 / tot : 0.0;  // no shift where the density vanishes
        double up[3];
        for (int d = 0; d < 3; ++d) up[d] = a[2 + d] - (F[0][d] + F[1][d]) * ih;
        for (int k = 0; k < 2; ++k) {
            double u[3];
            const bool ok = rho[k] >= 1e-12;  // no shift for a vanishing component
            for (int d = 0; d < 3; ++d) u[d] = ok ? up[d] + L.tau[k] * F[k][d] / rho[k] : up[d];
            const double usq = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
            for (int i = 0; i < Q; ++i) {
                const double cu = cx(i) * u[0] + cy(i) * u[1] + cz(i) * u[2];
                const double feq = wgt<double>(i) * rho[k] * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * usq);
                f[(k * Q + i) * L.fs + n] = Codec<S>::enc(typename Codec<S>::C(feq - wgt<double>(i) * L.rref[k]));
            }
        }
    }
}

int grid_for(int64_t n) {
    const int64_t g = (n + 255) / 256;
    return int(g < 1 ? 1 : (g > 8192 ? 8192 : g));
}

}  // namespace

// Which kernel a forward (DG = false) or input-gradient layer runs on:
//  * up to 32 or 64 columns on volumes of whole bricks: conv_brick (an input
//    gradient with fewer than 128 such work-groups goes on: 4 096 positions, 128 ->
//    64: 35 us against 13);
//  * where the GEMM's tiles would not fill the chip and K is long enough to be cut
//    into parts (forward: only with the layer's scratch acc, whose presence says
//    that K may be cut): conv_small, or conv_split where conv_small's work-groups
//    would come in more than two rounds, which is the line: 4 096 positions, 256 ->
//    128 (1 024 work-groups of 16 columns): 30 us, conv_split 43; 4 185 positions
//    (1 280): 45 and 43; 29 295 positions, 64 -> 64: 36 and 24.  Up to 32 columns
//    always conv_small (29 295 positions, 256 -> 32: 56 and 67).  Tiles of 128
//    where that leaves half the CUs at work (29 295 positions, 96 -> 128: 44 us,
//    tiles of 64 58; 12 480 positions: 42 and 31).
//    Layers of a network (ordered) take their parts from the size of a GEMM over
//    up to 512 work-groups and add them in one order, whichever kernel runs: a
//    BF16 network amplifies every other order of its early sums to 0.3 percent of
//    its output.  conv_split has up to four such parts; with so few of them half of
//    conv_small's wavefronts or more have nothing to do (28 672 positions, 192 ->
//    64: 184 us, conv_split 53; 64 -> 64: 49 and 24; at the line, 12 480 positions,
//    32 -> 64: 16 and 11);
//  * otherwise the GEMM (262 144 positions, 32 -> 96: 104 us, conv_small 190).
template <bool DG>
static hipError_t launch_conv(const ConvArgs &a, bool split, const uint16_t *g, float *dx, hipStream_t s) {
    const int P = a.D * a.H * a.W, N = DG ? a.c1 + a.c2 : a.cout, kc = DG ? a.cout : a.c1 + a.c2;
    const int nxy = (a.H / BRY) * (a.W / BRX);
    if (a.H % BRY == 0 && a.W % BRX == 0 && !(DG && N > 32 && nxy * (a.D / 2) < 128)) {
        if (N <= 32 && a.D % 4 == 0) {
            hipLaunchKernelGGL((conv_brick_kernel<4, 1, DG>), dim3(unsigned(nxy * (a.D / 4))), dim3(256), 0, s, a, g, dx);
            return hipGetLastError();
        }
        if (N <= 64 && a.D % 2 == 0) {
            hipLaunchKernelGGL((conv_brick_kernel<2, 2, DG>), dim3(unsigned(nxy * (a.D / 2))), dim3(256), 0, s, a, g, dx);
            return hipGetLastError();
        }
    }
    // 256-row tiles while they give at least ~2 work-groups per CU, else 128
    const int bn = N <= 32 ? 32 : (N <= 64 ? 64 : 128);
    const unsigned ny = unsigned((N + bn - 1) / bn);
    const bool big = int64_t((P + 255) / 256) * ny >= 512;
    const unsigned gx = unsigned(big ? (P + 255) / 256 : (P + 127) / 128);
    // parts of K: at least eight steps each, over up to 512 work-groups
    const int nst = (27 * kc + BK - 1) / BK, tiles = int(gx * ny);
    const int gz = split && tiles < 256 ? std::min(nst / 8, 512 / tiles) : 1;
    if (gz > 1) {
        const int nb = ((a.W + SBX - 1) / SBX) * ((a.H + SBY - 1) / SBY) * ((a.D + SBZ - 1) / SBZ);
        const int wgs = nb * ((N + 15) / 16);  // conv_small's work-groups of 16 columns
        const bool aligned = kc % BK == 0 && (DG || a.c1 % BK == 0);
        auto cut = [&](auto kern, int T, int KS) {
            const dim3 grid(unsigned((P + T - 1) / T), unsigned((N + T - 1) / T));
            hipLaunchKernelGGL(kern, grid, dim3(unsigned(256 * KS)), 0, s, a, g, dx);
            return hipGetLastError();
        };
        if (aligned && N > 32) {
            if (a.ordered && gz <= 4 && int64_t(wgs) * nst >= 40000)
                return gz == 2   ? cut(conv_split_kernel<64, 2, DG>, 64, 2)
                       : gz == 3 ? cut(conv_split_kernel<64, 3, DG>, 64, 3)
                                 : cut(conv_split_kernel<64, 4, DG>, 64, 4);
            if (!a.ordered && wgs >= 1100)
                return N > 64 && tiles >= 130 ? cut(conv_split_kernel<128, 2, DG>, 128, 2)
                                              : cut(conv_split_kernel<64, 3, DG>, 64, 3);
        }
        const int parts = a.ordered && kc % 32 == 0 && kc <= 256 ? gz : 0;
        // two column tiles per work-group share the halo and each LDS operand (four
        // spill with the parts' sums); one where that leaves CUs idle.  us with one /
        // two by work-groups of two: 128 -> 128 channels 7.6 / 10.3 with 64, 10.8 /
        // 10.5 with 168, 11.0 / 10.9 with 256, 19.7 / 17.4 with 512; 128 -> 256 7.7 /
        // 10.3 with 128, 19.1 / 16.6 with 512: even from 168 to 400, 192 taken
        const bool wide = nb * ((N + 31) / 32) >= 192;
        const dim3 grid(unsigned(nb), unsigned(wide ? (N + 31) / 32 : (N + 15) / 16));
        auto run = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(512), 0, s, a, g, dx, parts); };
        if (parts && kc > 128)
            wide ? run(conv_small_kernel<2, DG, 256>) : run(conv_small_kernel<1, DG, 256>);
        else
            wide ? run(conv_small_kernel<2, DG, 128>) : run(conv_small_kernel<1, DG, 128>);
        return hipGetLastError();
    }
    const dim3 grid(gx, ny);
    auto gemm = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, a, g, dx); };
    if (N <= 32)
        big ? gemm(conv_gemm_kernel<256, 32, 4, 1, DG>) : gemm(conv_gemm_kernel<128, 32, 4, 1, DG>);
    else if (N <= 64)
        big ? gemm(conv_gemm_kernel<256, 64, 4, 1, DG>) : gemm(conv_gemm_kernel<128, 64, 2, 2, DG>);
    else
        big ? gemm(conv_gemm_kernel<256, 128, 2, 2, DG>) : gemm(conv_gemm_kernel<128, 128, 2, 2, DG>);
    return hipGetLastError();
}

hipError_t launch_conv_fwd(const ConvArgs &a, bool split, hipStream_t s) {
    return launch_conv<false>(a, split, nullptr, nullptr, s);
}

hipError_t launch_conv_dgrad(const ConvArgs &a, const uint16_t *g, float *dx, hipStream_t s) {
    return launch_conv<true>(a, true, g, dx, s);
}

hipError_t launch_conv_wgrad(const ConvArgs &a, const uint16_t *g, float *dw, float *db, hipStream_t s) {
    const int nb = ((a.W + BRX - 1) / BRX) * ((a.H + BRY - 1) / BRY) * ((a.D + 3) / 4);
    const int ncb = (a.c1 + a.c2 + 31) / 32, nob = (a.cout + 31) / 32;
    // the bricks shared out over about WG_TARGET work-groups (two fit a CU, 512 the
    // chip): fewer leave CUs idle, more run in a second wave and add their sums into
    // dw more often.  us of a network's 15 layers with 256 / 384 / 448 / 512 / 640:
    // canvas 32 x 64 x 128 450 / 413 / 407 / 424 / 556; 32 x 56 x 128 420 / 397 / 399 /
    // 400 / 538; 40 x 72 x 136 664 / 570 / 577 / 562 / 776; 24 x 40 x 104 290 / 305 /
    // 303 / 316 / 411; 16 x 32 x 64 178 / 196 / 196 / 201 / 215; smaller ones even
    constexpr int WG_TARGET = 448;
    const int share = std::max(1, std::min(nb, WG_TARGET / (3 * ncb * nob)));
    hipLaunchKernelGGL(conv_wgrad_kernel, dim3(unsigned(share), unsigned(3 * ncb), unsigned(nob)), dim3(256), 0, s, a, g,
                       dw, db);
    return hipGetLastError();
}

hipError_t launch_pack_weights(PackList ls, hipStream_t s) {
    int tiles = 0;
    for (int L = 0; L < ls.n; ++L) {
        ls.at[L].tile0 = tiles;
        tiles += ((ls.at[L].K + 63) / 64) * ((ls.at[L].cout + 63) / 64);
    }
    hipLaunchKernelGGL(pack_weights_kernel, dim3(unsigned(tiles)), dim3(256), 0, s, ls);
    return hipGetLastError();
}

static bool aligned16(std::initializer_list<const void *> ps) {
    for (const void *p : ps)
        if (reinterpret_cast<uintptr_t>(p) & 15) return false;
    return true;
}

hipError_t launch_relu_grad(const float *dy, const uint16_t *y, int64_t n, int relu, uint16_t *g, hipStream_t s) {
    if (n % 8 == 0 && aligned16({dy, relu ? y : nullptr, g}))
        hipLaunchKernelGGL(relu_grad_kernel<8>, dim3(grid_for(n / 8)), dim3(256), 0, s, dy, y, n, relu, g);
    else
        hipLaunchKernelGGL(relu_grad_kernel<1>, dim3(grid_for(n)), dim3(256), 0, s, dy, y, n, relu, g);
    return hipGetLastError();
}

// the volume whose elements a pass of V channels per thread runs over: the
// coarser one (fine: the finer one) of D x H x W
static Vol vol_of(int D, int H, int W, int C, int V, bool fine) {
    Vol v;
    v.D = D / 2;
    v.H = H / 2;
    v.W = W / 2;
    v.C = C;
    v.n = (fine ? int64_t(D) * H * W : int64_t(v.D) * v.H * v.W) * (C / V);
    v.w = fine ? W : v.W;
    v.h = fine ? H : v.H;
    v.by_c = Divider(C / V);
    v.by_w = Divider(v.w);
    v.by_h = Divider(v.h);
    return v;
}

hipError_t launch_pool2(const uint16_t *x, int D, int H, int W, int C, uint16_t *y, hipStream_t s) {
    const int V = C % 8 == 0 && aligned16({x, y}) ? 8 : 1;
    const Vol v = vol_of(D, H, W, C, V, false);
    const dim3 grid(grid_for(v.n)), block(256);
    if (V == 8) hipLaunchKernelGGL(pool2_kernel<8>, grid, block, 0, s, x, v, y);
    else hipLaunchKernelGGL(pool2_kernel<1>, grid, block, 0, s, x, v, y);
    return hipGetLastError();
}

hipError_t launch_pool2_back(const float *gc, const float *skip, int skip_stride, int skip_off, int D, int H, int W,
                             int C, const uint16_t *my, float *g, uint16_t *gb, hipStream_t s) {
    const bool wide = C % 8 == 0 && skip_stride % 4 == 0 && skip_off % 4 == 0 && aligned16({gc, skip, my, g, gb});
    const Vol v = vol_of(D, H, W, C, wide ? 8 : 1, true);
    const dim3 grid(grid_for(v.n)), block(256);
    auto run = [&](auto k) { hipLaunchKernelGGL(k, grid, block, 0, s, gc, skip, skip_stride, skip_off, v, my, g, gb); };
    if (wide) run(pool2_back_kernel<8>);
    else run(pool2_back_kernel<1>);
    return hipGetLastError();
}

hipError_t launch_up2_back(const float *g, int stride, int C, int D, int H, int W, const uint16_t *my, float *gc,
                           uint16_t *gb, hipStream_t s) {
    const bool wide = C % 8 == 0 && stride % 4 == 0 && aligned16({g, my, gc, gb});
    const Vol v = vol_of(D, H, W, C, wide ? 8 : 1, false);
    const dim3 grid(grid_for(v.n)), block(256);
    auto run = [&](auto k) { hipLaunchKernelGGL(k, grid, block, 0, s, g, stride, v, my, gc, gb); };
    if (wide) run(up2_back_kernel<8>);
    else run(up2_back_kernel<1>);
    return hipGetLastError();
}

hipError_t launch_fill_f32(float *p, int64_t n, float v, hipStream_t s) {
    hipLaunchKernelGGL(fill_f32_kernel, dim3(grid_for(n)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_to_bf16(const float *x, int64_t n, uint16_t *y, hipStream_t s) {
    hipLaunchKernelGGL(to_bf16_kernel, dim3(grid_for(n)), dim3(256), 0, s, x, n, y);
    return hipGetLastError();
}

hipError_t launch_normalize(const float *x, int64_t P, const ChanScale &shift, const ChanScale &gain, uint16_t *y,
                            hipStream_t s) {
    hipLaunchKernelGGL(normalize_kernel, dim3(grid_for(P * 8)), dim3(256), 0, s, x, P, shift, gain, y);
    return hipGetLastError();
}

hipError_t launch_residual(const float *out, const float *xin, int64_t P, const ChanScale &sc, float *pred,
                           uint16_t *predb, hipStream_t s) {
    hipLaunchKernelGGL(residual_kernel, dim3(grid_for(P * 8)), dim3(256), 0, s, out, xin, P, sc, pred, predb);
    return hipGetLastError();
}

hipError_t launch_loss(const float *out, const float *xin, const float *tgt, int64_t P, const ChanScale &sc, double lam,
                       double *part, double *res, float *grad, hipStream_t s) {
    hipLaunchKernelGGL(loss_partial_kernel, dim3(LOSS_BLOCKS), dim3(256), 0, s, out, xin, tgt, P, sc, part);
    hipLaunchKernelGGL(loss_total_kernel, dim3(1), dim3(64), 0, s, part, LOSS_BLOCKS, lam, res);
    if (grad)
        hipLaunchKernelGGL(loss_grad_kernel, dim3(grid_for(P * 8)), dim3(256), 0, s, out, xin, tgt, P, sc, lam, res, grad);
    return hipGetLastError();
}

hipError_t launch_moments(const float *x, const float *y, int64_t P, double *part, double *res, hipStream_t s) {
    hipLaunchKernelGGL(moments_kernel, dim3(LOSS_BLOCKS), dim3(256), 0, s, x, y, P, part);
    hipLaunchKernelGGL(moments_total_kernel, dim3(1), dim3(64), 0, s, part, LOSS_BLOCKS, res);
    return hipGetLastError();
}

hipError_t launch_adam(float *p, const float *g, float *m, float *v, uint16_t *pb, int64_t n, int step, float lr, float b1,
                       float b2, float eps, hipStream_t s) {
    const float c1 = 1.0f - powf(b1, float(step)), c2 = 1.0f - powf(b2, float(step));
    hipLaunchKernelGGL(adam_kernel, dim3(grid_for(n)), dim3(256), 0, s, p, g, m, v, pb, n, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

template <class F>
static hipError_t by_prec(int prec, F &&fn) {
    switch (prec) {
        case LB_F64:
            return fn(static_cast<double *>(nullptr));
        case LB_F32:
            return fn(static_cast<float *>(nullptr));
        case LB_F16DEV:
            return fn(static_cast<_Float16 *>(nullptr));
        case LB_BF16DEV:
            return fn(static_cast<bf16_t *>(nullptr));
        default:
            return hipErrorInvalidValue;
    }
}

hipError_t launch_restrict(int prec, const void *f, const SurLattice &L, int D, int H, int W, float *outf,
                           uint16_t *outb, hipStream_t s) {
    const int gn = grid_for(int64_t(L.nx) * L.ny * L.nz), gc = (grid_for(8 * int64_t(D) * H * W) + 7) & ~7;
    return by_prec(prec, [&](auto *tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        const S *fs = static_cast<const S *>(f);
        hipLaunchKernelGGL(psi_state_kernel<S>, dim3(gn), dim3(256), 0, s, fs, L);
        hipLaunchKernelGGL(restrict_kernel, dim3(gc), dim3(256), 0, s, L, D, H, W, outf, outb);
        return hipGetLastError();
    });
}

hipError_t launch_lift(int prec, const float *coarse, int D, int H, int W, const SurLattice &L, void *f, hipStream_t s) {
    (void)D;
    const int64_t n_all = int64_t(L.nx) * L.ny * L.nz;
    const int gn = grid_for(n_all);
    // the block totals and the two factors follow psi in the scratch buffer
    // (the other population buffer: 2 Q fs elements of at least 2 bytes,
    // against 8 (2 n_all + 2 gn + 2) bytes here)
    double *part = L.psi + 2 * n_all;
    double *scale = part + 2 * gn;
    if ((2 * n_all + 2 * int64_t(gn) + 2) * 8 > 2 * int64_t(Q) * L.fs * 2) return hipErrorInvalidValue;
    return by_prec(prec, [&](auto *tag) {
        using S = std::remove_pointer_t<decltype(tag)>;
        hipLaunchKernelGGL(lift_mass_kernel, dim3(gn), dim3(256), 0, s, coarse, H, W, L, part);
        hipLaunchKernelGGL(lift_scale_kernel, dim3(1), dim3(256), 0, s, coarse, H, W, L, part, gn, scale);
        hipLaunchKernelGGL(psi_lift_kernel, dim3(gn), dim3(256), 0, s, coarse, H, W, L, scale);
        hipLaunchKernelGGL(lift_kernel<S>, dim3(gn), dim3(256), 0, s, coarse, H, W, L, scale, static_cast<S *>(f));
        return hipGetLastError();
    });
}

}  // namespace lbm
