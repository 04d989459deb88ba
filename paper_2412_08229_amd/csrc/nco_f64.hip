// NCO stream-collide of float64 lattices: the invariant network in float64
// on the matrix cores (v_mfma_f64_16x16x4), for every width, activation and
// depth.
//
// The same scheme as the float32 matrix-core network (nco_mfma.hip): tiles
// of 16 nodes as transposed GEMMs (hidden x nodes), the eight reflections of
// an axis permutation as a Walsh-Hadamard transform of eight parity-class
// products, each layer's accumulator the next layer's B operand.  The float64
// product's accumulator holds, in lane (q, c) = (lane / 16, lane % 16),
// element i = row 4 i + q of column c, so K-step ks of the next product takes
// hidden units 4 ks + q straight from element ks % 4 of tile ks / 4, and a
// width W (a multiple of 4) needs W / 4 K-steps and activates only its own
// rows, without padding.
//
// What bounds it: the float64 tanh (1,536 wavefront evaluations per 16-node
// tile at width 32, 24 instructions each) and then the products (148
// per axis permutation, 64 cycles each).  One tile per wavefront and four
// per block, so that a 40^3 lattice gives each SIMD four wavefronts; the
// weights of the products come from LDS (read by every wavefront of the
// block, 10 B/cycle), which leaves the registers to the 64 pre-activations
// of a permutation.  A 40^3 step of the 27-32-32-4 tanh network: 19.4 ms on
// the vector units (one lane per node, all weights unrolled: 8 KB of scratch
// per lane), 0.262 ms here.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "fold.h"
#include "kernels.h"
#include "stream.h"

namespace nco {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int F64_NODES = 64, F64_THREADS = 256;
constexpr int ROW64 = 29;           // LDS doubles per node: 27 moments, 1.0, 0.0

// Table of one network (doubles): per lane the A operands of the first layer
// [t MT][st 10][lane 64] and of each hidden-to-hidden layer [u MT][ks KS][lane
// 64]; then by row the biases of the hidden-to-hidden layers [W] each, W3 / 48
// [W][4] and b3 [4].
constexpr int mt_of(int W) { return (W + 15) / 16; }
constexpr int t64_a1(int) { return 0; }
constexpr int t64_a2(int W) { return mt_of(W) * KSTEPS * 64; }
constexpr int t64_a2b(int W) { return t64_a2(W) + mt_of(W) * (W / 4) * 64; }
constexpr int t64_b2(int W, int depth) { return t64_a2b(W) + (depth == 3 ? mt_of(W) * (W / 4) * 64 : 0); }
constexpr int t64_b2b(int W, int depth) { return t64_b2(W, depth) + W; }
constexpr int t64_w3(int W, int depth) { return t64_b2b(W, depth) + (depth == 3 ? W : 0); }
constexpr int t64_b3(int W, int depth) { return t64_w3(W, depth) + 4 * W; }
constexpr int t64_doubles(int W, int depth) { return t64_b3(W, depth) + 4; }

__device__ __forceinline__ f64x4 mfma64(double a, double b, f64x4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// tanh(z) = (2^y - 1) / (2^y + 1), y = 2 log2(e) z the pre-activation as the
// tables scale it; with n the nearest integer to y, f = y - n in [-1/2, 1/2] and
// c = 2^-n, numerator and denominator times c are (2^f - 1) + (1 - c) and that
// plus 2 c.  2^f - 1 = f P(f), P the interpolant of degree 10 of (2^f - 1) / f at
// the Chebyshev nodes (relative error 5.1e-17 with these rounded coefficients):
// no digits are lost near z = 0.  The reciprocal takes one step of third order
// from the hardware's estimate (24 bits).  Within 5 units of the last place.
// -n is capped so that c stays finite, after a conversion that is defined for
// every argument (the instruction saturates, where a cast leaves 2^31 and beyond
// undefined); an infinite y has the fraction 0 (infinity minus infinity would
// make it NaN, and tanh is +-1 there); a NaN stays NaN.  Clamping y itself cost
// 9 % of a step, this 1 %.
template <int ACT>
__device__ __forceinline__ double act64(double y) {
    if constexpr (ACT == ACT_RELU) {
        return y > 0.0 ? y : 0.0;
    } else {
        const double m = __builtin_rint(-y);
        double f = y + m;
        if (__builtin_isinf(y)) f = __hiloint2double(0, __double2loint(f));
        int k;
        asm("v_cvt_i32_f64 %0, %1" : "=v"(k) : "v"(m));
        double p = 4.4549605981865186e-10;
        p = fma(p, f, 7.072585949269223e-09);
        p = fma(p, f, 1.0178062445845774e-07);
        p = fma(p, f, 1.321544258792169e-06);
        p = fma(p, f, 1.525273382983612e-05);
        p = fma(p, f, 1.540353044173605e-04);
        p = fma(p, f, 1.3333558146416936e-03);
        p = fma(p, f, 9.618129107606888e-03);
        p = fma(p, f, 5.55041086648216e-02);
        p = fma(p, f, 2.4022650695910097e-01);
        p = fma(p, f, 6.931471805599453e-01);
        const double c = __builtin_amdgcn_ldexp(1.0, min(k, 1000));
        const double num = fma(p, f, 1.0 - c), d = fma(2.0, c, num);
        const double r = __builtin_amdgcn_rcp(d), e = fma(-d, r, 1.0);
        return num * fma(r, fma(e, e, e), r);
    }
}

// One hidden-to-hidden layer: c[u] = A h + b for the activations h[ks]
// (hidden unit 4 ks + q), A [u][ks] of this lane in LDS.
template <int W>
__device__ __forceinline__ void layer64(const double* __restrict__ a, const double* __restrict__ b, int lane, int q,
                                        const double (&h)[W / 4], f64x4 (&c)[mt_of(W)]) {
    constexpr int MT = mt_of(W), KS = W / 4;
#pragma unroll
    for (int u = 0; u < MT; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) c[u][i] = 4 * u + i < KS ? b[16 * u + 4 * i + q] : 0.0;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int u = 0; u < MT; ++u) c[u] = mfma64(a[(u * KS + ks) * 64 + lane], h[ks], c[u]);
}

// The rates of one 16-node tile (mrow: the moment row of the lane's node, sg:
// the gather table, tab: the network's table, both in LDS) to sw_node[4],
// written by the lanes of group q = 0.
template <int W, int ACT, int DEPTH>
__device__ __forceinline__ void network_f64(const double* __restrict__ mrow, const int* __restrict__ sg,
                                            const double* __restrict__ tab, int lane, double* __restrict__ sw_node) {
    constexpr int MT = mt_of(W), KS = W / 4;
    const int q = lane >> 4;
    double acc[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) acc[k] = 0.0;
#pragma unroll 1
    for (int p = 0; p < 6; ++p) {
        const int* __restrict__ ge = sg + (p * 4 + q) * GT_STRIDE;
        f64x4 Y[8][MT];
#pragma unroll
        for (int ci = 0; ci < 8; ++ci)
#pragma unroll
            for (int t = 0; t < MT; ++t) Y[ci][t] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int st = 0; st < KSTEPS; ++st) {
            const double b = mrow[ge[st]];
#pragma unroll
            for (int t = 0; t < MT; ++t)
                Y[step_class(st)][t] = mfma64(tab[t64_a1(W) + (t * KSTEPS + st) * 64 + lane], b, Y[step_class(st)][t]);
        }
#pragma unroll
        for (int bit = 1; bit < 8; bit <<= 1)
#pragma unroll
            for (int ci = 0; ci < 8; ++ci)
                if (!(ci & bit))
#pragma unroll
                    for (int k = 0; k < KS; ++k) {
                        const double u0 = Y[ci][k / 4][k % 4], u1 = Y[ci | bit][k / 4][k % 4];
                        Y[ci][k / 4][k % 4] = u0 + u1;
                        Y[ci | bit][k / 4][k % 4] = u0 - u1;
                    }
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            double h[KS];
            f64x4 c[MT];
#pragma unroll
            for (int k = 0; k < KS; ++k) h[k] = act64<ACT>(Y[s][k / 4][k % 4]);
            layer64<W>(tab + t64_a2(W), tab + t64_b2(W, DEPTH), lane, q, h, c);
            if constexpr (DEPTH == 3) {
#pragma unroll
                for (int k = 0; k < KS; ++k) h[k] = act64<ACT>(c[k / 4][k % 4]);
                layer64<W>(tab + t64_a2b(W), tab + t64_b2b(W, DEPTH), lane, q, h, c);
            }
#pragma unroll
            for (int k = 0; k < KS; ++k) acc[k] += act64<ACT>(c[k / 4][k % 4]);
        }
    }
    double pn[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        double v = 0.0;
#pragma unroll
        for (int k = 0; k < KS; ++k) v = fma(tab[t64_w3(W, DEPTH) + (4 * k + q) * 4 + n], acc[k], v);
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
        pn[n] = v;
    }
    if (q == 0)
#pragma unroll
        for (int n = 0; n < 4; ++n) sw_node[n] = squash_rate(pn[n] + tab[t64_b3(W, DEPTH) + n]);
}

// RATES: the rates of the stored state to omega_out [4][n] instead of a step.
template <int W, int ACT, int DEPTH, bool RATES>
__global__ __launch_bounds__(F64_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void k_nco_f64(
    const double* __restrict__ fin, double* __restrict__ fout, StepArgs a, const double* __restrict__ gtab_f64,
    double* __restrict__ omega_out) {
    constexpr int TAB = t64_doubles(W, DEPTH);
    __shared__ double tab[TAB];
    __shared__ double sm[F64_NODES * ROW64];
    __shared__ double sw[F64_NODES * 4];
    __shared__ int sg[GT_ENTRIES];
    const int tid = threadIdx.x;
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int idx = blk * F64_NODES + tid;
    for (int e = tid; e < TAB; e += F64_THREADS) tab[e] = gtab_f64[e];
    const int* __restrict__ gather = reinterpret_cast<const int*>(gtab_f64 + TAB);
    for (int e = tid; e < GT_ENTRIES; e += F64_THREADS) sg[e] = gather[e];
    const bool live = tid < F64_NODES && idx < a.n;
    if (tid < F64_NODES) {
        double f[Q], m[Q];
        if (live) {
            if constexpr (RATES)
                load_local<ST_F64>(fin, a.n, idx, f);
            else
                pull<ST_F64>(fin, a, node_of(idx, a.nx, a.ny), f);
        } else {
#pragma unroll
            for (int i = 0; i < Q; ++i) f[i] = weight_of(i);
        }
        to_moments(f, m);
        double* row = sm + tid * ROW64;
#pragma unroll
        for (int k = 0; k < Q; ++k) row[k] = m[row_tensor(k)];
        row[27] = 1.0;
        row[28] = 0.0;
    }
    __syncthreads();
    {
        const int lane = tid & 63, node = (tid >> 6) * 16 + (lane & 15);
        network_f64<W, ACT, DEPTH>(sm + node * ROW64, sg, tab, lane, sw + node * 4);
    }
    __syncthreads();
    if (!live) return;
    double omega[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) omega[n] = sw[tid * 4 + n];
    if constexpr (RATES) {
#pragma unroll
        for (int n = 0; n < 4; ++n) omega_out[(size_t)n * a.n + idx] = omega[n];
        return;
    }
    double f[Q], m[Q], dm[Q], df[Q];
    pull<ST_F64>(fin, a, node_of(idx, a.nx, a.ny), f);
    const double* row = sm + tid * ROW64;
#pragma unroll
    for (int k = 0; k < Q; ++k) m[row_tensor(k)] = row[k];
    if (a.n_modes > 0) {
        double Fx, Fy, Fz;
        read_force(a, idx, Fx, Fy, Fz);
        collision_delta<double, true>(m, a.omega_nu, omega, Fx, Fy, Fz, dm);
    } else {
        collision_delta<double, false>(m, a.omega_nu, omega, 0.0, 0.0, 0.0, dm);
    }
    from_moments(dm, df);
#pragma unroll
    for (int i = 0; i < Q; ++i) f[i] -= df[i];
    store_local<ST_F64>(fout, a.n, idx, f);
}

template <int W, int ACT, int DEPTH>
hipError_t launch_f64(const double* in, double* out, const StepArgs& a, const double* tab, double* omega_out,
                      hipStream_t st) {
    const dim3 grid((a.n + F64_NODES - 1) / F64_NODES), block(F64_THREADS);
    if (omega_out)
        hipLaunchKernelGGL((k_nco_f64<W, ACT, DEPTH, true>), grid, block, 0, st, in, out, a, tab, omega_out);
    else
        hipLaunchKernelGGL((k_nco_f64<W, ACT, DEPTH, false>), grid, block, 0, st, in, out, a, tab, omega_out);
    return hipGetLastError();
}

}  // namespace

size_t nco_f64_table_bytes(int width, int depth) {
    return sizeof(double) * t64_doubles(width, depth) + sizeof(int) * GT_ENTRIES;
}

void nco_f64_prepare_table(const float* params, int W, int act, int depth, const int (*gsrc)[27], void* out) {
    const float* W1 = params;
    const float* b1 = W1 + 27 * W;
    const float* W2 = b1 + W;
    const float* b2 = W2 + W * W;
    const float* W2b = b2 + W;                      // depth 3 only
    const float* b2b = W2b + W * W;
    const float* W3 = depth == 3 ? b2b + W : b2 + W;
    const float* b3 = W3 + 4 * W;
    const double kappa = act == ACT_TANH ? 2.0 / 0.69314718055994530942 : 1.0;
    const int MT = mt_of(W), KS = W / 4;
    double* tab = static_cast<double*>(out);
    int slot_row[KSTEPS][4];
    class_slots(slot_row);
    auto w1 = [&](int k, int h) { return k < 0 || h >= W ? 0.0 : (double)(k < 27 ? W1[k * W + h] : b1[h]); };
    auto hidden = [&](const float* w, const float* b, double* A, double* bias) {
        for (int u = 0; u < MT; ++u)
            for (int ks = 0; ks < KS; ++ks)
                for (int lane = 0; lane < 64; ++lane) {
                    const int in = 4 * ks + (lane >> 4), o = 16 * u + (lane & 15);
                    A[(u * KS + ks) * 64 + lane] = o < W ? kappa * w[in * W + o] : 0.0;
                }
        for (int o = 0; o < W; ++o) bias[o] = kappa * b[o];
    };
    for (int t = 0; t < MT; ++t)
        for (int st = 0; st < KSTEPS; ++st)
            for (int lane = 0; lane < 64; ++lane)
                tab[t64_a1(W) + (t * KSTEPS + st) * 64 + lane] =
                    kappa * w1(slot_row[st][lane >> 4], 16 * t + (lane & 15));
    hidden(W2, b2, tab + t64_a2(W), tab + t64_b2(W, depth));
    if (depth == 3) hidden(W2b, b2b, tab + t64_a2b(W), tab + t64_b2b(W, depth));
    for (int o = 0; o < W; ++o)
        for (int n = 0; n < 4; ++n) tab[t64_w3(W, depth) + o * 4 + n] = (double)W3[o * 4 + n] / NGROUP;
    for (int n = 0; n < 4; ++n) tab[t64_b3(W, depth) + n] = b3[n];
    int* gtab = reinterpret_cast<int*>(tab + t64_doubles(W, depth));
    for (int p = 0; p < 6; ++p)
        for (int q = 0; q < 4; ++q)
            for (int i = 0; i < GT_STRIDE; ++i) {
                const int k = i < KSTEPS ? slot_row[i][q] : -1;
                gtab[(p * 4 + q) * GT_STRIDE + i] = k < 0 ? 28 : k == 27 ? 27 : gsrc[8 * p][k];
            }
}

hipError_t launch_nco_f64(const void* fin, void* fout, const StepArgs& a, const void* table, double* omega_out,
                          hipStream_t st) {
    const double* in = static_cast<const double*>(fin);
    double* out = static_cast<double*>(fout);
    const double* tab = static_cast<const double*>(table);
#define F64_CASE(WW, DD)                                                                                   \
    if (a.width == WW && a.depth == DD)                                                                    \
        return a.act == ACT_TANH ? launch_f64<WW, ACT_TANH, DD>(in, out, a, tab, omega_out, st)            \
                                 : launch_f64<WW, ACT_RELU, DD>(in, out, a, tab, omega_out, st);
    // Depth 3 runs at width 32 (narrower networks are zero-padded).
    F64_CASE(8, 2) F64_CASE(16, 2) F64_CASE(20, 2) F64_CASE(32, 2) F64_CASE(32, 3)
#undef F64_CASE
    return hipErrorInvalidValue;
}

}  // namespace nco
