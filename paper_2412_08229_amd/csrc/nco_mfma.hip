// Operand tables of the matrix-core networks, the choice of arithmetic, and
// the float32 network's kernels.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "nco_mfma.h"

namespace nco {

NCO_NET_DEFINE(f32, MLP_PREC_F32)

namespace {

unsigned bf16_bits(float v) {                 // round to nearest even
    unsigned u;
    std::memcpy(&u, &v, 4);
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

float bf16_value(unsigned bits) {
    const unsigned u = bits << 16;
    float v;
    std::memcpy(&v, &u, 4);
    return v;
}

unsigned f16_bits(float v) {                  // round to nearest even (the compiler's conversion)
    const _Float16 h = (_Float16)v;
    unsigned short u;
    std::memcpy(&u, &h, 2);
    return u;
}

}  // namespace

size_t mfma_lane_table_floats() { return 64 * LANE_WORDS; }
size_t mfma_group_table_ints() { return GT_ENTRIES; }

// Host-side preparation of the per-lane operand table from the flat
// parameters (W1[27][W], b1, W2[W][W], b2, W3[W][4], b3) and of the gather
// table: for axis permutation p and K slot holding W1 row k, the moment row
// that m^(g) places at k.  gsrc is indexed by group element g = 8 p +
// reflection mask; the reflection-free elements g = 8 p give Q_p.
void mfma_prepare_tables(const float* params, int act, int prec, const int (*gsrc)[27], float* lane_tab,
                         int* gtab, int depth, int units) {
    const int W = MW;
    const bool u20 = units <= 20;
    const float* W1 = params;
    const float* b1 = W1 + 27 * W;
    const float* W2 = b1 + W;
    const float* b2 = W2 + W * W;
    const float* W2b = b2 + W;                      // depth 3 only
    const float* b2b = W2b + W * W;
    const float* W3 = depth == 3 ? b2b + W : b2 + W;
    const float* b3 = W3 + 4 * W;
    const bool th = act == ACT_TANH && prec != MLP_PREC_F32_FULL;
    const float kappa = th ? (float)(2.0 / 0.69314718055994530942) : 1.0f;
    // tanh = 1 - 2 r folded into the consumer of each activation:
    // W2 -> -2 W2, b2 -> b2 + sum_h W2[h][:], W3 -> -2 W3, b3 -> b3 + sum_h W3[h][:]
    // (the group mean turns 1 into 48 / 48).
    const float fold = th ? -2.0f : 1.0f;
    float b2f[MW], b3f[4];
    for (int o = 0; o < W; ++o) {
        double s = b2[o];
        if (th)
            for (int h = 0; h < W; ++h) s += W2[h * W + o];
        b2f[o] = (float)s;
    }
    for (int n = 0; n < 4; ++n) {
        double s = b3[n];
        if (th)
            for (int h = 0; h < W; ++h) s += W3[h * 4 + n];
        b3f[n] = (float)s;
    }
    auto w1row = [&](int k, int h) { return k < 27 ? W1[k * W + h] : k == 27 ? b1[h] : 0.0f; };
    // Split arithmetic, tanh: per layer (first, second, third) the power of
    // two sigma that puts the largest |A| (kappa W1 with the bias row, kappa
    // fold W2, kappa fold W2b) into [128, 256), well inside the f16 range,
    // with the remainders of all but negligible weights normal; b2bf the
    // third layer's bias with the tanh fold.
    float split_sigma[3] = {1.0f, 1.0f, 1.0f};
    float b2bf[MW] = {};
    if (prec == MLP_PREC_F32S && th) {
        float amax[3] = {0.0f, 0.0f, 0.0f};
        for (int k = 0; k < 28; ++k)
            for (int h = 0; h < W; ++h) amax[0] = std::max(amax[0], std::fabs(kappa * w1row(k, h)));
        for (int i = 0; i < W * W; ++i) {
            amax[1] = std::max(amax[1], std::fabs(kappa * fold * W2[i]));
            if (depth == 3) amax[2] = std::max(amax[2], std::fabs(kappa * fold * W2b[i]));
        }
        for (int l = 0; l < 3; ++l)
            if (amax[l] > 0.0f) split_sigma[l] = std::ldexp(1.0f, 7 - std::ilogb(amax[l]));
    }
    if (depth == 3)
        for (int o = 0; o < W; ++o) {
            double sb = b2b[o];
            if (th)
                for (int h = 0; h < W; ++h) sb += W2b[h * W + o];
            b2bf[o] = (float)sb;
        }
    int slot_row[KSTEPS][4];
    class_slots(slot_row);
    for (int lane = 0; lane < 64; ++lane) {
        const int q = lane >> 4, c = lane & 15;
        const LaneTabT<float> lt(lane_tab, lane);
        const LaneTabT<unsigned> lw(reinterpret_cast<unsigned*>(lane_tab), lane);
        for (int i = 0; i < LANE_WORDS; ++i) lt[i] = 0.0f;
        // Unit in row c of tile t, and in row 4 q + r as K slot or
        // accumulator; weights of hidden-to-hidden layers between them.
        auto row = [&](int t) { return tile_unit(u20, t, c / 4, c % 4); };
        auto slot = [&](int t, int r) { return tile_unit(u20, t, q, r); };
        auto hidden = [&](const float* Wl, int u, int t, int r) {
            return row(u) < 0 || slot(t, r) < 0 ? 0.0f : kappa * fold * Wl[slot(t, r) * W + row(u)];
        };
        auto first = [&](int k, int t) { return k < 0 || row(t) < 0 ? 0.0f : kappa * w1row(k, row(t)); };
        auto bias = [&](const float* b, int u, int r) { return slot(u, r) < 0 ? 0.0f : kappa * b[slot(u, r)]; };
        if (prec == MLP_PREC_F32S) {
            // Parts of each layer's A operand in the K slots of its product:
            // layer 1 slot j of lane group q holds input row 8 q + j, a
            // hidden-to-hidden layer's slot j the hidden unit of tile j / 4,
            // row 4 q + j % 4.
            auto put = [&](int off, int t, int w, int e, float a) {
                unsigned part[3];
                if (th) {
                    part[0] = f16_bits(a);
                    part[1] = f16_bits(a - (float)(_Float16)a);
                    part[2] = 0;
                } else {
                    part[0] = bf16_bits(a);
                    const float r = a - bf16_value(part[0]);
                    part[1] = bf16_bits(r);
                    part[2] = bf16_bits(r - bf16_value(part[1]));
                }
                for (int k = 0; k < 3; ++k) lw[off + 12 * t + 4 * k + w] |= part[k] << (16 * e);
            };
            if (th) {
                for (int t = 0; t < 2; ++t)
                    for (int w = 0; w < 4; ++w)
                        for (int e = 0; e < 2; ++e)
                            put(LS_A1, t, w, e, split_sigma[0] * first(8 * q + 2 * w + e, t));
                lt[LS_BACK] = 1.0f / split_sigma[0];
            } else {
                for (int t = 0; t < 2; ++t)
                    for (int st = 0; st < KSTEPS; ++st) lt[LT_A1 + t * KSTEPS + st] = first(slot_row[st][q], t);
            }
            auto fill = [&](const float* Wl, const float* bfold, float sigma, int offA, int offB, int slot) {
                for (int u = 0; u < 2; ++u)
                    for (int w = 0; w < 4; ++w)
                        for (int e = 0; e < 2; ++e)
                            put(offA, u, w, e, sigma * hidden(Wl, u, w / 2, 2 * (w % 2) + e));
                const float up = th ? sigma * 2048.0f : 1.0f;
                for (int u = 0; u < 2; ++u)
                    for (int r = 0; r < 4; ++r) lt[offB + u * 4 + r] = up * bias(bfold, u, r);
                lt[LS_BACK + slot] = 1.0f / up;
            };
            fill(W2, b2f, split_sigma[1], LS_A2, LS_B2, 1);
            if (depth == 3) fill(W2b, b2bf, split_sigma[2], LS_A3, LS_B3, 2);
            lt[LS_NEG1] = -1.0f;
            for (int b = 0; b < 3; ++b)
                for (int w = 0; w < 4; ++w) {
                    const int k0 = 8 * q + 2 * w, k1 = k0 + 1;
                    lw[LS_SM + 4 * b + w] = ((row_class(k0) >> b) & 1 ? 0x8000u : 0u) |
                                            ((row_class(k1) >> b) & 1 ? 0x80000000u : 0u);
                }
            for (int u = 0; u < 2; ++u)
                for (int r = 0; r < 4; ++r)
                    for (int n = 0; n < 4; ++n)
                        lt[LS_W3 + (u * 4 + r) * 4 + n] = fold * W3[(16 * u + 4 * q + r) * 4 + n] / (float)NGROUP;
            for (int n = 0; n < 4; ++n) lt[LS_B3O + n] = b3f[n];
        } else if (prec == MLP_PREC_F32 || prec == MLP_PREC_F32_FULL) {
            for (int t = 0; t < 2; ++t)
                for (int st = 0; st < KSTEPS; ++st) lt[LT_A1 + t * KSTEPS + st] = first(slot_row[st][q], t);
            for (int u = 0; u < 2; ++u)
                for (int t = 0; t < 2; ++t)
                    for (int r = 0; r < 4; ++r) lt[LT_A2 + u * 8 + t * 4 + r] = hidden(W2, u, t, r);
            for (int u = 0; u < 2; ++u)
                for (int r = 0; r < 4; ++r) lt[LT_B2 + u * 4 + r] = bias(b2f, u, r);
            for (int u = 0; u < 2; ++u)
                for (int r = 0; r < 4; ++r)
                    for (int n = 0; n < 4; ++n)
                        lt[LT_W3 + (u * 4 + r) * 4 + n] = fold * W3[(16 * u + 4 * q + r) * 4 + n] / (float)NGROUP;
            for (int n = 0; n < 4; ++n) lt[LT_B3 + n] = b3f[n];
            if (depth == 3) {
                // Third layer: tanh of the second folded in as for W2 above.
                for (int v = 0; v < 2; ++v)
                    for (int t = 0; t < 2; ++t)
                        for (int r = 0; r < 4; ++r) lt[LT_A2B + v * 8 + t * 4 + r] = hidden(W2b, v, t, r);
                for (int v = 0; v < 2; ++v)
                    for (int r = 0; r < 4; ++r) lt[LT_B2B + v * 4 + r] = bias(b2bf, v, r);
            }
        } else {
            // K slot j of lane group q is row k = 8 q + j (layer 1) and the
            // hidden unit of tile j / 4, row 4 q + j % 4.
            auto pair = [](float x0, float x1) { return bf16_bits(x0) | (bf16_bits(x1) << 16); };
            auto layer = [&](const float* Wl, const float* b, int offA, int offB) {
                for (int u = 0; u < 2; ++u) {
                    for (int w = 0; w < 4; ++w)
                        lw[offA + 4 * u + w] =
                            pair(hidden(Wl, u, w / 2, 2 * (w % 2)), hidden(Wl, u, w / 2, 2 * (w % 2) + 1));
                    for (int r = 0; r < 4; ++r) lt[offB + u * 4 + r] = bias(b, u, r);
                }
            };
            for (int t = 0; t < 2; ++t)
                for (int w = 0; w < 4; ++w)
                    lw[LB_A1 + 4 * t + w] = pair(first(8 * q + 2 * w, t), first(8 * q + 2 * w + 1, t));
            layer(W2, b2f, LB_A2, LB_B2);
            // Third layer, in the second's layout, tanh of the second folded
            // in as for W2.
            if (depth == 3) layer(W2b, b2bf, LB_A2B, LB_B2B);
            for (int u = 0; u < 2; ++u)
                for (int r = 0; r < 4; ++r)
                    for (int n = 0; n < 4; ++n)
                        lt[LB_W3 + (u * 4 + r) * 4 + n] = fold * W3[(16 * u + 4 * q + r) * 4 + n] / (float)NGROUP;
            for (int n = 0; n < 4; ++n) lt[LB_B3 + n] = b3f[n];
            for (int b = 0; b < 3; ++b)
                for (int w = 0; w < 4; ++w) {
                    const int k0 = 8 * q + 2 * w, k1 = k0 + 1;
                    lw[LB_SM + 4 * b + w] = ((row_class(k0) >> b) & 1 ? 0x8000u : 0u) |
                                            ((row_class(k1) >> b) & 1 ? 0x80000000u : 0u);
                }
        }
    }
    for (int p = 0; p < 6; ++p)
        for (int q = 0; q < 4; ++q)
            for (int i = 0; i < GT_STRIDE; ++i) {
                // Row k placed in this slot; 27 is the constant-1 row, 28 zero.
                int k = -1;
                if (prec == MLP_PREC_F32 || prec == MLP_PREC_F32_FULL || (prec == MLP_PREC_F32S && !th)) {
                    if (i < KSTEPS) k = slot_row[i][q];
                } else if (i < 8) {
                    k = 8 * q + i;
                }
                int e = 28;
                if (k >= 0 && k < 27) e = gsrc[8 * p][k];
                if (k == 27) e = 27;
                gtab[(p * 4 + q) * GT_STRIDE + i] = e;
            }
}

// omega_out == nullptr: one stream-collide step fin -> fout.  Otherwise the
// rates of the state in fin are written to omega_out and fout is untouched.
hipError_t launch_nco_mfma(int storage, int prec, const void* fin, void* fout, const StepArgs& a,
                           const float* lane_tab, const int* gtab, double* omega_out, hipStream_t st) {
    switch (prec) {
        case MLP_PREC_F32_FULL: return launch_net_full(storage, fin, fout, a, lane_tab, gtab, omega_out, st);
        case MLP_PREC_BF16: return launch_net_bf16(storage, fin, fout, a, lane_tab, gtab, omega_out, st);
        case MLP_PREC_F32S: return launch_net_split(storage, fin, fout, a, lane_tab, gtab, omega_out, st);
        default: return launch_net_f32(storage, fin, fout, a, lane_tab, gtab, omega_out, st);
    }
}

hipError_t launch_nco_mfma_grouped(int storage, int prec, int act, int units, const LaunchGroup& g, hipStream_t st) {
    switch (prec) {
        case MLP_PREC_BF16: return launch_net_bf16_grouped(storage, act, units, g, st);
        case MLP_PREC_F32S: return launch_net_split_grouped(storage, act, units, g, st);
        default: return launch_net_f32_grouped(storage, act, units, g, st);
    }
}

}  // namespace nco
