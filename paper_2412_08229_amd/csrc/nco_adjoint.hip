// Reverse mode of one step with a matrix-core network (float32, depth 2 or
// 3): given lambda = dL/dx_t+1, the pre-collision adjoint M^T g_m + lambda is
// scattered back along the streaming, and the parameter gradient of this
// step is added to the block's row of `partial` (float64, one row per block,
// each row touched by its block only, so the sum over steps is in a fixed
// order).  The same computation as the vector-unit adjoint (adjoint.hip).
//
// Per node tile of 16 and group element g = (pi, s), in the layout of the
// forward network (hidden x nodes, lane (q, c) = (lane / 16, lane % 16)
// holding rows 4 q .. 4 q + 3 of node c):
//   forward recompute   r_l = act(Z_l)
//   dz_L = dh_L (.) act'(z_L),   dh_L = W3 dtt / 48 (the same for every g)
//   dh_l-1 = W_l dz_l,   dz_l-1 = dh_l-1 (.) act'(z_l-1)   (products whose
//         B operands are the previous accumulators, as in the forward)
//   dW_l += h_l-1 dz_l^T, db_l += dz_l                      (products over the
//         16 nodes of the tile)
// and per permutation, with Z_cl = sum_s chi_s(cl) dz1_s over its 8
// reflections (Walsh-Hadamard transform) for the 8 parity classes of W1's
// rows:
//   dL/dm[src_pi(k)] += (W1 Z_class(k))[k],   dW1[k] += x_pi[k] Z_class(k)^T
// (the bias row of x_pi gives db1).
// For tanh at depth 2, with r = 1 / (1 + 2^(kappa z)): h = 1 - 2 r, act' =
// 4 r (1 - r); the 4 is folded into the transposed weights and W3 (exactly, a
// power of 2).  At depth 3 tanh itself on the unfolded weights, act' = 1 - h^2:
// h = 1 - 2 r is right to 6e-8 of one, and the gradient of a layer fed by small
// activations would be no better than that over their size.  The group sum H
// of the output layer's gradient is added up here as well, not unfolded from
// the forward step's.  It costs 17-25 % of a reverse step: 16^3 63 -> 74 us,
// 64^3 1707 -> 2139.
//
// Products over nodes.  h and dz go through a per-wavefront LDS buffer
// [hidden][node] of row stride 20: a lane reads the nodes 4 q .. 4 q + 3 of
// one hidden unit in one 16-byte read, which makes step st of the product
// node 4 q + st for both operands; the rows of 8 lanes of a read fall on
// distinct banks.
//
// Products per class.  The classes have 9 (with the bias row), 4, 4, 4, 2, 2,
// 2 and 1 rows: ten groups of up to four rows, each with its own Z.  They run
// on 4x4x1 products of 16 independent blocks, two row groups at a time (five
// pairs): dW1 as (row group 2) x (hidden 32 / 4), one node per product; dL/dm as
// (half of the hidden units 2) x (row group 2) x (nodes 16 / 4), one hidden
// unit per half and product.  160 products of 8 cycles per permutation and
// tile, where 16x16x4 products with four classes per tile took 128 of 32.
//
// What bounds it: the matrix cores and the vector instructions share a pipe
// in float32; at depth 2 a permutation of a tile is 404 products of 32 cycles
// and 160 of 8 beside 256 transcendentals and ~1,300 other vector
// instructions.  The weights are read from LDS, not held in registers, which
// lets two wavefronts share a SIMD (256 registers) and fill each other's
// waits; with the weights in registers (490) one wavefront per SIMD ran.
//
// Measured per reverse step with kept network values, before (weights in
// registers at depth 2, vector units at depth 3) and here: depth 2 tanh 16^3
// 105 -> 47 us, 32^3 203 -> 154, 64^3 1390 -> 1078, 96^3 4870 -> 3640 (about
// 60 TFLOP/s of products, 40 % of what a large float32 product reaches);
// depth 3 tanh 16^3 348 -> 74, 32^3 1537 -> 288, 64^3 11960 -> 2139.
//
// Networks of at most 20 hidden units (depth 3) lie in the tiles as in the
// forward step (act_tail): five K-steps and activations instead of eight; the
// products over nodes and per class stay (rows without a unit are zero or not
// read).  Width 20, ReLU: 16^3 61 -> 52 us, 32^3 219 -> 175, 64^3 1606 -> 1264.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "adjoint.h"
#include "net_f32.h"
#include "stream.h"

namespace nco {

namespace {

constexpr int PAIRS = 5;
constexpr int TSTRIDE = 20;                   // row stride of the transpose buffers
constexpr int TBUF = 32 * TSTRIDE;

// Parity classes of the row groups, two groups per pair.
__host__ __device__ constexpr int pair_class(int a, int g) {
    constexpr int c[PAIRS][2] = {{0, 0}, {0, 1}, {2, 4}, {3, 5}, {6, 7}};
    return c[a][g];
}

// Table of the reverse step, the same for all blocks (copied to LDS): floats,
// then ints.
constexpr int TA_A1 = 0;                      // [t 2][st 10][lane 64]      W1 rows / b1 as A operand
constexpr int TA_A2 = TA_A1 + 1280;           // [u 2][t 2][lane 64][r 4]   W2 as A operand
constexpr int TA_W2T = TA_A2 + 1024;          // [t 2][u 2][lane 64][r 4]   W2[16 t + c][16 u + 4 q + r]
constexpr int TA_W1 = TA_W2T + 1024;          // [pair][half 2][group 2][row 4][16] W1[row][16 half + .] (no row: 0)
constexpr int TA_B2 = TA_W1 + 1280;           // [32] accumulator init of layer 2
constexpr int TA_W3F = TA_B2 + 32;            // [32][4] W3 / 48, folded for the forward pass
constexpr int TA_B3F = TA_W3F + 128;          // [4]
constexpr int TA_W3 = TA_B3F + 4;             // [32][4] W3 / 48 (times 4 for tanh)
constexpr int TA_A2B = TA_W3 + 128;           // depth 3: as A2, W2T and B2 of the third layer
constexpr int TA_W2BT = TA_A2B + 1024;
constexpr int TA_B2B = TA_W2BT + 1024;
constexpr int ta_floats(int depth) { return depth == 3 ? TA_B2B + 32 : TA_A2B; }
constexpr int TI_GE = 0;                      // [p 6][q 4][GT_STRIDE] moment rows of the K slots
constexpr int TI_SRC = GT_ENTRIES;            // [p 6][pair][8] moment row src_pi(row) (27: bias, 28: no row)
constexpr int TI_ROW = TI_SRC + 6 * PAIRS * 8;   // [pair][8] row of M (27: bias, 28: none)
constexpr int TI_INTS = TI_ROW + PAIRS * 8;

__device__ __forceinline__ f32x4 mfma4x4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0);
}

// Only one wavefront's LDS words are exchanged: order, no block barrier.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// act' (for the folded tanh without its 4) and h from the activation r.
template <int ACT>
__device__ __forceinline__ float act_slope(float r) {
    return act_base(ACT) == ACT_RELU ? (r > 0.0f ? 1.0f : 0.0f)
                                     : fmaf(-r, r, act_base(ACT) == ACT_TANH_FULL ? 1.0f : r);
}
template <int ACT>
__device__ __forceinline__ float act_value(float r) {
    return act_base(ACT) == ACT_TANH ? fmaf(-2.0f, r, 1.0f) : r;
}

__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// v (hidden 16 t + 4 q + r of node c) to buf [hidden][node]; of the second
// tile the first TAIL rows of each lane.
template <int TAIL = 4>
__device__ __forceinline__ void to_buf(float* __restrict__ buf, int q, int c, const f32x4 (&v)[2]) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < (t == 0 ? 4 : TAIL); ++r) buf[(16 * t + 4 * q + r) * TSTRIDE + c] = v[t][r];
}

// g[x][y] += sum over the tile's nodes of h[16 x + .] dz[16 y + .]^T, through
// the two buffers (rows that hold no unit give entries that are not read).
template <int TAIL>
__device__ __forceinline__ void outer_product(float* __restrict__ buf, int q, int c, const f32x4 (&h)[2],
                                              const f32x4 (&dz)[2], f32x4 (&g)[2][2]) {
    to_buf<TAIL>(buf, q, c, h);
    to_buf<TAIL>(buf + TBUF, q, c, dz);
    wave_sync();
    f32x4 a[2], b[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        a[x] = ld4(buf + (16 * x + c) * TSTRIDE + 4 * q);
        b[x] = ld4(buf + TBUF + (16 * x + c) * TSTRIDE + 4 * q);
    }
    wave_sync();
#pragma unroll
    for (int st = 0; st < 4; ++st)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) g[x][y] = mfma4(a[x][st], b[y][st], g[x][y]);
}

// WAVES = 4: 64 nodes at a time, `groups` times, one 16-node tile per
// wavefront, its six axis permutations in series.  WAVES = 6 (small lattices):
// one tile, one permutation per wavefront (a sixth of the chain, and a block
// per 16 nodes).
template <int S, int ACT, int DEPTH, int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(2))) void k_adjoint_net(
    const typename Codec<S>::store_t* __restrict__ xin, const float* __restrict__ lam_in, float* __restrict__ lam_out,
    StepArgs a, const float* __restrict__ table, double* __restrict__ partial, int groups) {
    constexpr int THREADS = 64 * WAVES;
    constexpr int TILES = WAVES == 4 ? 4 : 1, NB = 16 * TILES, NS = NB + 4;
    constexpr int COPIES = WAVES == 4 ? 1 : WAVES;      // dL/dm sums in LDS
    constexpr int TAF = ta_floats(DEPTH);
    constexpr int ROW = DEPTH == 3 ? NPAR3 : NPAR;
    constexpr bool FULL = act_base(ACT) == ACT_TANH_FULL;
    constexpr int FWD = FULL ? ACT - ACT_TANH_FULL + ACT_TANH : ACT;    // the forward step's activation
    __shared__ __align__(16) float tab[TAF + TI_INTS];
    __shared__ __align__(16) float sm[29 * NS];         // [moment row][node]; row 27 = 1, 28 = 0
    __shared__ float sdm[COPIES == 1 ? 32 * NS : COPIES * 29 * NS];   // group sums [32][node], then dL/dm
    __shared__ float sgm[Q * NS];                       // the collision's part of dL/dm
    __shared__ float sw[4 * NS];                        // tilde tau, then dL/d tilde tau
    __shared__ __align__(16) float bufs[WAVES][2 * TBUF];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, q = lane >> 4, c = lane & 15;
    const int* __restrict__ ti = reinterpret_cast<const int*>(tab + TAF);
    static_assert((TAF + TI_INTS) % 4 == 0, "the table is copied in 16-byte pieces");
    for (int e = 4 * tid; e < TAF + TI_INTS; e += 4 * THREADS)
        *reinterpret_cast<f32x4*>(tab + e) = *reinterpret_cast<const f32x4*>(table + e);
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    float* __restrict__ buf = bufs[wave];

    f32x4 gW1[PAIRS], gW2[2][2], gW2b[2][2], gb2[2], gb2b[2];
#pragma unroll
    for (int k = 0; k < PAIRS; ++k) gW1[k] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        gb2[x] = gb2b[x] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int y = 0; y < 2; ++y) gW2[x][y] = gW2b[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    constexpr int TAIL = act_tail(ACT);
    double gW3 = 0.0;                                   // entry tid of W3, then of b3 (tid < 132)

    // wl: the lane's place in the weight tables, hidden from the compiler anew
    // for every group element (fresh_lane): the weights are read from LDS where
    // they are used instead of being kept in registers.
    int wl = lane;
    auto A1 = [&](int t, int st) { return tab[TA_A1 + (t * KSTEPS + st) * 64 + lane]; };
    auto A2 = [&](int u, int t, int r) { return tab[TA_A2 + ((u * 2 + t) * 64 + wl) * 4 + r]; };
    auto W2T = [&](int t, int u, int r) { return tab[TA_W2T + ((t * 2 + u) * 64 + wl) * 4 + r]; };
    auto A2b = [&](int v, int t, int r) { return tab[TA_A2B + ((v * 2 + t) * 64 + wl) * 4 + r]; };
    auto W2bT = [&](int t, int v, int r) { return tab[TA_W2BT + ((t * 2 + v) * 64 + wl) * 4 + r]; };
    // A row vector of 32 floats as the accumulator rows of this lane.
    auto rows = [&](int off, f32x4(&v)[2]) {
#pragma unroll
        for (int u = 0; u < 2; ++u) v[u] = ld4(tab + off + 16 * u + 4 * q);
    };

    for (int grp = 0; grp < groups; ++grp) {
        const int first = (blk * groups + grp) * NB;
        if (first >= a.n) break;
        const int idx = first + tid;
        const bool live = tid < NB && idx < a.n;
        __syncthreads();
        // Phase A: moments of the pulled state.  In a tile the pulls (with
        // their folds at the faces of the reduced cube) are shared by all
        // threads (16^3 depth 3 with the scatter: 62 -> 50 us a step); a
        // thread of a 64-node block pulls its node (64^3 shared: 1.5 % slower).
        if constexpr (WAVES != 4) {
            for (int e = tid; e < Q * NB; e += THREADS) {
                const int i = e / NB, nd = e % NB;
                sgm[i * NS + nd] = first + nd < a.n ? pull_one<S>(xin, a, node_of(first + nd, a.nx, a.ny), i)
                                                    : (float)weight_of(i);
            }
            __syncthreads();
        }
        if (tid < NB) {
            float f[Q], m[Q];
            if constexpr (WAVES != 4) {
#pragma unroll
                for (int i = 0; i < Q; ++i) f[i] = sgm[i * NS + tid];
            } else if (live) {
                pull<S>(xin, a, node_of(idx, a.nx, a.ny), f);
            } else {
#pragma unroll
                for (int i = 0; i < Q; ++i) f[i] = (float)weight_of(i);
            }
            to_moments(f, m);
#pragma unroll
            for (int k = 0; k < Q; ++k) sm[k * NS + tid] = m[row_tensor(k)];
            sm[27 * NS + tid] = 1.0f;
            sm[28 * NS + tid] = 0.0f;
        }
        // Phase B1: group sums (unless they come from phase B3) and tilde tau,
        // kept by the forward step of this state (places past the last node
        // read as zero) or computed again, the same arithmetic in the same order.
        if (a.net_sums) {
            for (int e = tid; e < NB * NET_SUMS_PER_NODE; e += THREADS) {
                const int nd = e / NET_SUMS_PER_NODE, k = e % NET_SUMS_PER_NODE;
                const float v = first + nd < a.n ? a.net_sums[(size_t)first * NET_SUMS_PER_NODE + e] : 0.0f;
                if (k >= 32)
                    sw[(k - 32) * NS + nd] = v;
                else if constexpr (!FULL)
                    sdm[k * NS + nd] = v;
            }
            __syncthreads();
        } else {
            __syncthreads();
            if (wave < TILES) {
                const int node = wave * 16 + c;
                f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
                // The forward step's weights: the table's, or its own where the
                // table holds the unfolded ones.
                const LaneTab lt(table + TAF + TI_INTS, lane);
                auto fA1 = [&](int t, int st) { return FULL ? lt[LT_A1 + t * KSTEPS + st] : A1(t, st); };
                auto fA2 = [&](int u, int t, int r) { return FULL ? lt[LT_A2 + u * 8 + t * 4 + r] : A2(u, t, r); };
                auto fA2b = [&](int v, int t, int r) { return FULL ? lt[LT_A2B + v * 8 + t * 4 + r] : A2b(v, t, r); };
                auto fB = [&](int off, int word, f32x4(&v)[2]) {
                    rows(off, v);
                    if constexpr (FULL)
#pragma unroll
                        for (int u = 0; u < 2; ++u)
#pragma unroll
                            for (int r = 0; r < 4; ++r) v[u][r] = lt[word + u * 4 + r];
                };
#pragma unroll 1
                for (int p = 0; p < 6; ++p) {
                    const int* __restrict__ ge = ti + TI_GE + (p * 4 + q) * GT_STRIDE;
                    f32x4 Y[8][2], b2[2], b2b[2];
                    layer1_f32<TAIL>(fA1, [&](int st) { return sm[ge[st] * NS + node]; }, Y);
                    reflections(Y);
                    fB(TA_B2, LT_B2, b2);
                    if constexpr (DEPTH == 3)
                        fB(TA_B2B, LT_B2B, b2b);
                    else
                        fB(TA_B2, LT_B2, b2b);
                    hidden_reflections<FWD, DEPTH, 8>(
                        fA2, b2, fA2b, b2b, Y, [&]() { fresh_lane(wl); },
                        [&](int, const f32x4(&z)[2]) { add_act<FWD>(z, acc); });
                }
                units_in_order<ACT>(acc, q, c);
                if constexpr (!FULL)
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int r = 0; r < 4; ++r) sdm[(16 * u + 4 * q + r) * NS + node] = acc[u][r];
                for (int n = 0; n < 4; ++n) {
                    float v = 0.0f;
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            v = fmaf(FULL ? lt[LT_W3 + (u * 4 + r) * 4 + n]
                                          : tab[TA_W3F + (16 * u + 4 * q + r) * 4 + n],
                                     acc[u][r], v);
                    v += __shfl_xor(v, 16, 64);
                    v += __shfl_xor(v, 32, 64);
                    if (q == 0) sw[n * NS + node] = v + (FULL ? lt[LT_B3 + n] : tab[TA_B3F + n]);
                }
            }
            __syncthreads();
        }
        // Phase B2: per node, the collision's part of dL/dm and dL/d tilde tau.
        if (tid < NB) {
            float m[Q], lam[Q], nu[Q], gm[Q], omega[4], tau[4], e[4], domega[4], F[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int i = 0; i < Q; ++i) lam[i] = live ? lam_in[(size_t)i * a.n + idx] : 0.0f;
            if (a.n_modes > 0 && live) read_force(a, idx, F[0], F[1], F[2]);
#pragma unroll
            for (int k = 0; k < Q; ++k) m[row_tensor(k)] = sm[k * NS + tid];
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                e[n] = expf(sw[n * NS + tid]);
                tau[n] = 0.5f + 0.5f / (1.0f + e[n]);
                omega[n] = 1.0f / tau[n];
            }
            inverse_T(lam, nu);
            collision_vjp_local(m, nu, a.omega_nu_f, omega, a.n_modes > 0, F, gm, domega);
#pragma unroll
            for (int k = 0; k < Q; ++k) sgm[k * NS + tid] = gm[row_tensor(k)];
#pragma unroll
            for (int n = 0; n < 4; ++n)
                sw[n * NS + tid] = domega[n] * 0.5f * e[n] / ((1.0f + e[n]) * (1.0f + e[n]) * tau[n] * tau[n]);
        }
        __syncthreads();
        // Output layer: dW3 = sum (H / 48) dtt^T with H the group sum of the
        // (unfolded) last-layer activations, db3 = sum dtt.
        auto output_gradient = [&](auto&& H) {
            if (tid < 132) {
                const int o = tid >> 2, n = tid & 3;        // o = 32: b3
                float v = 0.0f;
                for (int nd = 0; nd < NB; ++nd) {
                    const float d = sw[n * NS + nd];
                    if (o < 32)
                        v = fmaf(H(o, nd) * (1.0f / NGROUP), d, v);
                    else
                        v += d;
                }
                gW3 += (double)v;
            }
        };
        if constexpr (!FULL)
            output_gradient([&](int o, int nd) {
                const float acc = sdm[o * NS + nd];
                return act_base(ACT) == ACT_RELU ? acc : (float)NGROUP - 2.0f * acc;
            });
        __syncthreads();
        for (int e = tid; e < COPIES * 29 * NS; e += THREADS) sdm[e] = 0.0f;
        __syncthreads();

        // Phase B3: the network adjoint.
        {
            const int base = WAVES == 4 ? wave * 16 : 0, node = base + c;
            float* __restrict__ dmc = sdm + (COPIES == 1 ? 0 : wave * 29 * NS);
            f32x4 dhl[2], hsum[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float v = 0.0f;
#pragma unroll
                    for (int n = 0; n < 4; ++n)
                        v = fmaf(tab[TA_W3 + (16 * u + 4 * q + r) * 4 + n], sw[n * NS + node], v);
                    dhl[u][r] = v;
                }
            // One permutation per wavefront of six: still a loop to the
            // compiler (which spilled 300 registers scheduling it as one
            // straight piece with what surrounds it).
            int p0 = WAVES == 4 ? 0 : __builtin_amdgcn_readfirstlane(wave), p1 = WAVES == 4 ? 6 : p0 + 1;
            if constexpr (WAVES != 4) asm volatile("" : "+s"(p1));
#pragma unroll 1
            for (int p = p0; p < p1; ++p) {
                const int* __restrict__ ge = ti + TI_GE + (p * 4 + q) * GT_STRIDE;
                // Pre-activations of the eight reflections; dz1 of reflection
                // s takes the place of Z[s] once they are used.
                f32x4 Z[8][2];
                layer1_f32<TAIL>(A1, [&](int st) { return sm[ge[st] * NS + node]; }, Z);
                reflections(Z);
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    f32x4 r1[2], r2[2], dz[2], h[2];
                    fresh_lane(wl);
                    act_f32<ACT>(Z[s], r1);
                    rows(TA_B2, h);
                    hidden_f32<TAIL>(A2, r1, h);
                    act_f32<ACT>(h, r2);
                    if constexpr (DEPTH == 3) {
                        f32x4 r3[2], v[2];
                        rows(TA_B2B, h);
                        hidden_f32<TAIL>(A2b, r2, h);
                        act_f32<ACT>(h, r3);
#pragma unroll
                        for (int u = 0; u < 2; ++u)
#pragma unroll
                            for (int r = 0; r < act_values(ACT, u); ++r) {
                                dz[u][r] = dhl[u][r] * act_slope<ACT>(r3[u][r]);
                                gb2b[u][r] += dz[u][r];
                                if constexpr (FULL) hsum[u][r] += r3[u][r];
                                v[u][r] = act_value<ACT>(r2[u][r]);
                            }
                        outer_product<TAIL>(buf, q, c, v, dz, gW2b);
                        h[0] = h[1] = f32x4{0.f, 0.f, 0.f, 0.f};
                        hidden_f32<TAIL>(W2bT, dz, h);
                    } else {
                        h[0] = dhl[0];
                        h[1] = dhl[1];
                    }
                    {
                        f32x4 v[2];
#pragma unroll
                        for (int u = 0; u < 2; ++u)
#pragma unroll
                            for (int r = 0; r < act_values(ACT, u); ++r) {
                                dz[u][r] = h[u][r] * act_slope<ACT>(r2[u][r]);
                                gb2[u][r] += dz[u][r];
                                v[u][r] = act_value<ACT>(r1[u][r]);
                            }
                        outer_product<TAIL>(buf, q, c, v, dz, gW2);
                    }
                    h[0] = h[1] = f32x4{0.f, 0.f, 0.f, 0.f};
                    hidden_f32<TAIL>(W2T, dz, h);
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            Z[s][t][r] = r < act_values(ACT, t) ? h[t][r] * act_slope<ACT>(r1[t][r]) : 0.0f;
                }
                reflections(Z);
                // The row groups of the classes, two at a time.
#pragma unroll
                for (int k = 0; k < PAIRS; ++k) {
                    const int c0 = pair_class(k, 0), c1 = pair_class(k, 1);
                    if (k != 1) to_buf(buf, q, c, Z[c0]);       // pair 1 keeps class 0 of pair 0
                    if (c1 != c0) to_buf(buf + TBUF, q, c, Z[c1]);
                    wave_sync();
                    const int* __restrict__ src = ti + TI_SRC + (p * PAIRS + k) * 8;
                    // dL/dm: lane (half, group, nodes 4 ng .., i).
                    {
                        const int half = lane >> 5, g = (lane >> 4) & 1, ng = (lane >> 2) & 3, i = lane & 3;
                        const float* __restrict__ w = tab + TA_W1 + (((k * 2 + half) * 2 + g) * 4 + i) * 16;
                        const float* __restrict__ z =
                            buf + (c1 != c0 && g ? TBUF : 0) + 16 * half * TSTRIDE + 4 * ng + i;
                        f32x4 D[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                        for (int j = 0; j < 16; j += 4) {
                            const f32x4 wv = ld4(w + j);
#pragma unroll
                            for (int e = 0; e < 4; ++e) D[e & 1] = mfma4x4(wv[e], z[(j + e) * TSTRIDE], D[e & 1]);
                        }
                        // Each half finishes two of the group's four rows.
                        const f32x4 d = D[0] + D[1];
                        const float x0 = half ? d[0] : d[2], x1 = half ? d[1] : d[3];
                        const float y0 = (half ? d[2] : d[0]) + __shfl_xor(x0, 32, 64);
                        const float y1 = (half ? d[3] : d[1]) + __shfl_xor(x1, 32, 64);
                        const int nd = base + 4 * ng + i, r0 = 4 * g + 2 * half;
                        dmc[src[r0] * NS + nd] += y0;
                        dmc[src[r0 + 1] * NS + nd] += y1;
                    }
                    // dW1: lane (group, hidden 4 cg .., i).
                    {
                        const int g = lane >> 5, cg = (lane >> 2) & 7, i = lane & 3;
                        const float* __restrict__ x = sm + src[4 * g + i] * NS + base;
                        const float* __restrict__ z = buf + (c1 != c0 && g ? TBUF : 0) + (4 * cg + i) * TSTRIDE;
#pragma unroll
                        for (int nd = 0; nd < 16; nd += 4) {
                            const f32x4 xv = ld4(x + nd), zv = ld4(z + nd);
#pragma unroll
                            for (int e = 0; e < 4; ++e) gW1[k] = mfma4x4(xv[e], zv[e], gW1[k]);
                        }
                    }
                    wave_sync();
                }
            }
            if constexpr (FULL) {
                units_in_order<ACT>(hsum, q, c);
                to_buf(buf, q, c, hsum);
            }
        }
        __syncthreads();
        // The group sum, from the wavefront of the node's tile or from the six
        // that share it.
        if constexpr (FULL)
            output_gradient([&](int o, int nd) {
                float v = bufs[nd >> 4][o * TSTRIDE + (nd & 15)];
                if constexpr (WAVES != 4)
                    for (int w = 1; w < WAVES; ++w) v += bufs[w][o * TSTRIDE + nd];
                return v;
            });
        if constexpr (COPIES > 1) {
            for (int e = tid; e < Q * NS; e += THREADS) {
                float t = sdm[e];
                for (int w = 1; w < COPIES; ++w) t += sdm[w * 29 * NS + e];
                sdm[e] = t;
            }
            __syncthreads();
        }
        // Phase C: the full collision adjoint per node, scattered along the
        // streaming.
        if (live) {
            float gm[Q], gf[Q], v[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i) v[i] = lam_in[(size_t)i * a.n + idx];
#pragma unroll
            for (int k = 0; k < Q; ++k) gm[row_tensor(k)] = sgm[k * NS + tid] + sdm[k * NS + tid];
            moments_T(gm, gf);
#pragma unroll
            for (int i = 0; i < Q; ++i) v[i] += gf[i];
            if constexpr (WAVES == 4) {
                scatter_to_sources(lam_out, a, node_of(idx, a.nx, a.ny), v);
            } else {
#pragma unroll
                for (int i = 0; i < Q; ++i) sgm[i * NS + tid] = v[i];
            }
        }
        if constexpr (WAVES != 4) {
            __syncthreads();
            for (int e = tid; e < Q * NB; e += THREADS) {
                const int i = e / NB, nd = e % NB;
                if (first + nd < a.n)
                    scatter_one(lam_out, a, node_of(first + nd, a.nx, a.ny), i, sgm[i * NS + nd]);
            }
        }
    }
    __syncthreads();

    // Block sums of the wavefronts' gradients, in wavefront order, added to
    // the block's row.
    double* __restrict__ out = partial + (size_t)blk * ROW;
    // One add per entry and launch (the block owns its row): an atomic without
    // return, so that the block does not wait for the row's old values.
    auto add = [&](int e, double v) { unsafeAtomicAdd(out + e, v); };
    float* __restrict__ red = &bufs[0][0];
    if (tid < 128)
        add(OFF_W3 + tid, gW3);
    else if (tid < 132)
        add(OFF_B3 + tid - 128, gW3);
    // The unit in row j of the 32 rows of a layer, -1 for none.
    auto unit = [](int j) { return tile_unit(TAIL == 1, j >> 4, (j >> 2) & 3, j & 3); };
    // A hidden-to-hidden layer: lane (q, c) holds [j = 16 x + 4 q + r][o = 16 y + c].
    auto add_layer = [&](const f32x4(&g)[2][2], const f32x4(&gb)[2], int offw, int offb) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int r = 0; r < 4; ++r) red[wave * 1024 + (16 * x + 4 * q + r) * 32 + 16 * y + c] = g[x][y][r];
        __syncthreads();
        for (int e = tid; e < 1024; e += THREADS) {
            const int j = unit(e >> 5), o = unit(e & 31);
            if (j < 0 || o < 0) continue;
            float v = red[e];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) v += red[w * 1024 + e];
            add(offw + j * 32 + o, (double)v);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[(wave * 16 + c) * 32 + 16 * u + 4 * q + r] = gb[u][r];
        __syncthreads();
        if (tid < 32 && unit(tid) >= 0) {
            float v = 0.0f;
            for (int w = 0; w < 16 * WAVES; ++w) v += red[w * 32 + tid];
            add(offb + unit(tid), (double)v);
        }
        __syncthreads();
    };
    add_layer(gW2, gb2, OFF_W2, OFF_B2);
    if constexpr (DEPTH == 3) add_layer(gW2b, gb2b, OFF_W2B, OFF_B2B);
    // dW1 and db1: lane (group, cg, i) holds [row r of the group][j = 4 cg + i].
#pragma unroll
    for (int k = 0; k < PAIRS; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            red[wave * (PAIRS * 256) + (k * 8 + (lane >> 5) * 4 + r) * 32 + (lane & 31)] = gW1[k][r];
    __syncthreads();
    for (int e = tid; e < PAIRS * 256; e += THREADS) {
        const int row = ti[TI_ROW + (e >> 5)], j = unit(e & 31);
        if (row > 27 || j < 0) continue;
        float v = red[e];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) v += red[w * (PAIRS * 256) + e];
        add(row < 27 ? OFF_W1 + row * 32 + j : OFF_B1 + j, (double)v);
    }
}

// Lattices up to this many nodes run one tile per six-wavefront block.  A
// block fills a CU's registers (two wavefronts on two of its SIMDs), so 256
// blocks run at a time, each two permutations long where a 64-node block's
// wavefronts run six in series; at two rounds (8192 nodes, depth 2) 79
// against 103 us, at four (24^3) the 64-node blocks are faster.
constexpr int ADJ_TILE_NODES = 8192;
// 64-node blocks take up to four groups of nodes one after another, so that
// fewer gradient rows are read and written per step, while the ~512 blocks
// that run at a time still have two each.
int adjoint_groups(int n) { return std::max(1, std::min(4, n / 65536)); }

}  // namespace

size_t mfma_adjoint_table_bytes(int depth) {
    return sizeof(float) * (ta_floats(depth) + (depth == 3 ? mfma_lane_table_floats() : 0)) + sizeof(int) * TI_INTS;
}

void mfma_prepare_adjoint_table(const float* params, int act, int depth, int units, const int (*gsrc)[27],
                                const float* folded, void* out) {
    const int W = MW;
    const bool u20 = units <= 20;
    auto weight = [&](const float* Wl, int j, int o) { return j < 0 || o < 0 ? 0.0f : Wl[j * W + o]; };
    const float* W1 = params;
    const float* b1 = W1 + 27 * W;
    const float* W2 = b1 + W;
    const float* b2 = W2 + W * W;
    const float* W2b = b2 + W;                      // depth 3 only
    const float* b2b = W2b + W * W;
    const float* W3 = depth == 3 ? b2b + W : b2 + W;
    float* tab = static_cast<float*>(out);
    int* ti = reinterpret_cast<int*>(tab + ta_floats(depth));
    // The forward weights in the order of the forward step's own table: its
    // very values, or with tanh at depth 3 the unfolded ones, behind which the
    // forward step's table follows.
    const bool full = act == ACT_TANH && depth == 3;
    const size_t nf = mfma_lane_table_floats(), ni = mfma_group_table_ints();
    std::vector<float> own(folded ? 0 : nf + ni), unfolded(full ? nf + ni : 0);     // floats, then ints
    auto build = [&](int prec, std::vector<float>& t) {
        mfma_prepare_tables(params, act, prec, gsrc, t.data(), reinterpret_cast<int*>(t.data() + nf), depth, units);
    };
    if (!folded) {
        build(MLP_PREC_F32, own);
        folded = own.data();
    }
    if (full) build(MLP_PREC_F32_FULL, unfolded);
    const float* fwd = full ? unfolded.data() : folded;
    const int* gather = reinterpret_cast<const int*>(folded + nf);
    if (depth == 3) std::memcpy(ti + TI_INTS, folded, sizeof(float) * nf);
    const float slope = act == ACT_TANH && !full ? 4.0f : 1.0f;
    for (int lane = 0; lane < 64; ++lane) {
        const LaneTab lt(fwd, lane);
        const int q = lane >> 4, c = lane & 15;
        for (int t = 0; t < 2; ++t)
            for (int st = 0; st < KSTEPS; ++st) tab[TA_A1 + (t * KSTEPS + st) * 64 + lane] = lt[LT_A1 + t * KSTEPS + st];
        for (int u = 0; u < 2; ++u)
            for (int t = 0; t < 2; ++t)
                for (int r = 0; r < 4; ++r) {
                    const int e = ((u * 2 + t) * 64 + lane) * 4 + r;
                    tab[TA_A2 + e] = lt[LT_A2 + u * 8 + t * 4 + r];
                    // Row c of tile u of the transposed layer's output, rows 4 q + r of tile t of its input.
                    const int j = tile_unit(u20, u, c / 4, c % 4), o = tile_unit(u20, t, q, r);
                    tab[TA_W2T + e] = slope * weight(W2, j, o);
                    if (depth == 3) {
                        tab[TA_A2B + e] = lt[LT_A2B + u * 8 + t * 4 + r];
                        tab[TA_W2BT + e] = slope * weight(W2b, j, o);
                    }
                }
        if (c == 0)
            for (int u = 0; u < 2; ++u)
                for (int r = 0; r < 4; ++r) {
                    const int row = 16 * u + 4 * q + r;
                    tab[TA_B2 + row] = lt[LT_B2 + u * 4 + r];
                    if (depth == 3) tab[TA_B2B + row] = lt[LT_B2B + u * 4 + r];
                    for (int n = 0; n < 4; ++n) tab[TA_W3F + row * 4 + n] = lt[LT_W3 + (u * 4 + r) * 4 + n];
                }
        if (lane == 0)
            for (int n = 0; n < 4; ++n) tab[TA_B3F + n] = lt[LT_B3 + n];
    }
    for (int j = 0; j < W; ++j)
        for (int n = 0; n < 4; ++n) {
            const int o = tile_unit(u20, j / 16, j / 4 % 4, j % 4);
            tab[TA_W3 + j * 4 + n] = o < 0 ? 0.0f : slope * (W3[o * 4 + n] / (float)NGROUP);
        }
    // Row groups: the rows of each class (the bias row 27 with class 0) in
    // groups of four, 28 where there is none.
    int taken[8] = {0};
    for (int k = 0; k < PAIRS; ++k)
        for (int g = 0; g < 2; ++g) {
            const int cl = pair_class(k, g);
            for (int i = 0; i < 4; ++i) {
                int seen = 0, row = 28;
                for (int r = 0; r < 28 && row == 28; ++r)
                    if (row_class(r) == cl && seen++ == taken[cl] + i) row = r;
                ti[TI_ROW + k * 8 + g * 4 + i] = row;
                for (int half = 0; half < 2; ++half)
                    for (int j = 0; j < 16; ++j)
                        tab[TA_W1 + (((k * 2 + half) * 2 + g) * 4 + i) * 16 + j] =
                            row < 27 ? weight(W1, row, tile_unit(u20, half, j / 4, j % 4)) : 0.0f;
                for (int p = 0; p < 6; ++p)
                    ti[TI_SRC + (p * PAIRS + k) * 8 + g * 4 + i] = row < 27 ? gsrc[8 * p][row] : row;
            }
            taken[cl] += 4;
        }
    for (int e = 0; e < GT_ENTRIES; ++e) ti[TI_GE + e] = gather[e];
}

int adjoint_mfma_blocks(int n) {
    if (n <= ADJ_TILE_NODES) return (n + 15) / 16;
    const int per = 64 * adjoint_groups(n);
    return (n + per - 1) / per;
}

hipError_t launch_adjoint_mfma(int storage, int act, const void* xin, const float* lam_in, float* lam_out,
                               const StepArgs& a, const void* table, double* partial, hipStream_t st) {
    const bool tile = a.n <= ADJ_TILE_NODES;
    const int groups = tile ? 1 : adjoint_groups(a.n);
    const dim3 grid(adjoint_mfma_blocks(a.n));
    const float* tab = static_cast<const float*>(table);
#define ADJN(SS, AA, DD, WW)                                                                          \
    hipLaunchKernelGGL((k_adjoint_net<SS, AA, DD, WW>), grid, dim3(64 * WW), 0, st,                   \
                       static_cast<const typename Codec<SS>::store_t*>(xin), lam_in, lam_out, a, tab, \
                       partial, groups)
#define ADJN_SHAPE(SS, AA, DD)       \
    if (tile) ADJN(SS, AA, DD, 6);   \
    else ADJN(SS, AA, DD, 4);
#define ADJN_CASE(SS)                                               \
    case SS:                                                        \
        if (a.depth == 3 && a.units <= 20) {                        \
            if (act == ACT_TANH) { ADJN_SHAPE(SS, ACT_TANH_FULL + UNITS_20, 3) } \
            else { ADJN_SHAPE(SS, ACT_RELU + UNITS_20, 3) }         \
        } else if (a.depth == 3) {                                  \
            if (act == ACT_TANH) { ADJN_SHAPE(SS, ACT_TANH_FULL, 3) } \
            else { ADJN_SHAPE(SS, ACT_RELU, 3) }                    \
        } else {                                                    \
            if (act == ACT_TANH) { ADJN_SHAPE(SS, ACT_TANH, 2) }    \
            else { ADJN_SHAPE(SS, ACT_RELU, 2) }                    \
        }                                                           \
        return hipGetLastError();
    switch (storage) {
        ADJN_CASE(ST_F32)
        ADJN_CASE(ST_F16)
        ADJN_CASE(ST_BF16)
        default: return hipErrorInvalidValue;
    }
#undef ADJN_CASE
#undef ADJN_SHAPE
#undef ADJN
}

}  // namespace nco
