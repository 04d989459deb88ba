// Kernels of the float32 network in full (nco_mfma.h): no folding, tanh
// itself.  A quarter of a hidden layer's products where the network has at most
// 16 hidden units (width 8, 64^3: 0.26 against 0.48 ms for tanh, 0.11 against
// 0.28 for ReLU).
//
// It replaces a vector-unit network, one lane per node and its 48 elements in
// series: width 32, tanh, depth 2 16^3 3.68 ms -> 17 us, 40^3 3.69 -> 0.15 ms,
// 64^3 11.8 -> 0.59; width 20, ReLU, depth 3 64^3 2.97 -> 0.31; width 8, ReLU
// 64^3 0.154 -> 0.108 - with the same errors of the rates against float64
// (root mean square 4.0e-8, largest 1.2e-7; the folded form: 4.2e-8, 1.5e-7).
#include "nco_mfma.h"

namespace nco {

namespace {

template <int S, int DD>
hipError_t launch_full(const void* fin, void* fout, const StepArgs& a, const float* lane_tab, const int* gtab,
                       double* omega_out, hipStream_t st) {
    constexpr int PP = MLP_PREC_F32;
    if (a.act == ACT_RELU) return launch_kind<S, ACT_RELU + UNITS_16, PP, DD>(fin, fout, a, lane_tab, gtab, omega_out, st);
    if (a.units <= 16)
        return launch_kind<S, ACT_TANH_FULL + UNITS_16, PP, DD>(fin, fout, a, lane_tab, gtab, omega_out, st);
    if (a.units <= 20)
        return launch_kind<S, ACT_TANH_FULL + UNITS_20, PP, DD>(fin, fout, a, lane_tab, gtab, omega_out, st);
    return launch_kind<S, ACT_TANH_FULL, PP, DD>(fin, fout, a, lane_tab, gtab, omega_out, st);
}

}  // namespace

hipError_t launch_net_full(int storage, const void* fin, void* fout, const StepArgs& a, const float* lane_tab,
                           const int* gtab, double* omega_out, hipStream_t st) {
    // ReLU has nothing to fold: the float32 network's kernels, but for their
    // smallest form.
    if (a.act == ACT_RELU && a.units > 16) return launch_net_f32(storage, fin, fout, a, lane_tab, gtab, omega_out, st);
#define NCO_STORAGE(SS)                                                                             \
    case SS:                                                                                        \
        return a.depth == 3 ? launch_full<SS, 3>(fin, fout, a, lane_tab, gtab, omega_out, st)       \
                            : launch_full<SS, 2>(fin, fout, a, lane_tab, gtab, omega_out, st);
    switch (storage) {
        NCO_STORAGE(ST_F32)
        NCO_STORAGE(ST_F16)
        NCO_STORAGE(ST_BF16)
        default: return hipErrorInvalidValue;
    }
#undef NCO_STORAGE
}

}  // namespace nco
