// NCO stream-collide with the invariant network on the matrix cores (gfx950).
//
// Network of Eq. gconv_m, evaluated for tiles of 16 nodes as transposed
// GEMMs (hidden x nodes):
//     Z1_g = W1^T m^(g) + b1     (32 x 28) (28 x 16)
//     H1   = act(Z1_g)
//     Z2_g = W2^T H1 + b2        (32 x 32) (32 x 16)
//     acc += act(Z2_g)           summed over the 48 elements g of O_h
//     tilde tau = W3^T acc / 48 + b3
// in one of these arithmetics:
//   F32_FULL  v_mfma_f32_16x16x4f32 (float32 operands and accumulation), tanh
//             itself;
//   F32       the same products, tanh folded into the weights (net_f32.h);
//   BF16      v_mfma_f32_16x16x32_bf16 (bf16 operands, float32 accumulation,
//             activations and group sum in float32);
//   F32S      float32 operands split into 16-bit parts, whose products run on
//             the f16 or bf16 matrix cores (split_layer).
//
// Group structure.  An element g of O_h is an axis permutation pi followed by
// axis reflections s in {+-1}^3.  Every row of M is a product of
// one-dimensional Hermite polynomials, so m^(g) = M Pi_g f is the permuted
// moment vector (Q_pi m) with row k multiplied by prod_r s_r^(n_kr): the sign
// depends only on the parity class c(k) = (n_kx, n_ky, n_kz) mod 2 of the row.
//  * float32: Z1_(pi,s) = sum_c chi_s(c) Y_(pi,c) with Y_(pi,c) =
//    W1_c^T (Q_pi m)_c and chi_s(c) = prod_r s_r^(c_r), i.e. the eight
//    reflections of one permutation are a 3-point Walsh-Hadamard transform of
//    eight class partial products (10 K-steps of 4 instead of 8 x 7).
//  * bf16: one K = 32 product covers all 28 rows, so each element is one
//    product per output tile; the reflection is applied to the packed bf16
//    operand by flipping sign bits with per-lane class masks.
// The moment operand is gathered from LDS once per permutation.
//
// Register chaining.  The accumulator of a 16x16 product holds, in lane
// (q, c) = (lane / 16, lane % 16), rows 4q..4q+3 of column c.  Ordering the K
// index of the next product as (t, r) -> hidden 16 t + 4 q + r (float32,
// K = 4 per step) or (j / 4, j % 4) -> hidden 16 (j / 4) + 4 q + j % 4 for the
// 8 K values j of a lane (bf16, K = 32) makes that exactly its B operand, so
// layer 2 consumes act(Z1) straight from registers.
//
// Block = 256 threads = 256 nodes.  Phase A: each thread pulls its 27
// populations and writes its 27 moments (plus the constant 1 of the bias row)
// to LDS.  Phase B: each wavefront runs the network for its 64 nodes, 16 at a
// time, and writes the four rates per node to LDS.  Phase C: each thread pulls
// its populations again (the kernel is compute bound; the second read is
// cheap), relaxes with the rates and stores.  Smaller lattices take other block
// shapes (launch_kind).
//
// One source per arithmetic instantiates the kernels (nco_mfma.hip float32,
// nco_mfma_full.hip float32 without the folding of tanh, nco_mfma_split.hip,
// nco_mfma_bf16.hip).
#pragma once

#include "kernels.h"
#include "net_f32.h"
#include "stream.h"

namespace nco {

namespace {

constexpr int NODE_STRIDE = 29;     // LDS floats per node: 27 moments, 1.0, 0.0

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// Split arithmetic (network_split): per layer the parts of its A operand as
// packed pairs in the K slots of the 16x16x32 product ([t or u 2][part 3][4
// words]: f16 head and remainder for tanh, bf16 head, middle and tail for
// ReLU; layer 1 of tanh in the slots of the bf16 path, K slot j of lane
// group q holding input row 8 q + j, layer 1 of ReLU as LT_A1 on the
// float32 matrix cores), the accumulator inits of the hidden-to-hidden
// layers, the scales that return each product to the pre-activation, the
// sign masks of the reflections and the output layer.
constexpr int LS_A1 = 0;
constexpr int LS_A2 = 24;
constexpr int LS_A3 = 48;
constexpr int LS_B2 = 72;           // [u 2][r 4]
constexpr int LS_B3 = 80;           // [u 2][r 4]
constexpr int LS_BACK = 88;         // [layer 1, 2, 3]
constexpr int LS_NEG1 = 91;         // -1.0 (see residual_f16)
constexpr int LS_SM = 92;           // [bit 3][4 words] as LB_SM
constexpr int LS_W3 = 104;          // [u 2][r 4][n 4] W3 / 48
constexpr int LS_B3O = 136;         // [n 4]
// bf16 path (A operands as packed bf16 pairs, two per word):
constexpr int LB_A1 = 0;            // [t 2][4 words]  W1 rows 8q..8q+7 / b1
constexpr int LB_A2 = 8;            // [u 2][4 words]  W2
constexpr int LB_B2 = 16;           // [u 2][r 4]
constexpr int LB_W3 = 24;           // [u 2][r 4][n 4]
constexpr int LB_B3 = 56;           // [n 4]
constexpr int LB_SM = 60;           // [bit 3][4 words] sign masks of classes with that bit
constexpr int LB_A2B = 72;          // [v 2][4 words]  W2b (depth 3)
constexpr int LB_B2B = 80;          // [v 2][r 4]      b2b (depth 3)

__device__ __forceinline__ f32x4 mfma32(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Two floats to a packed bf16 pair (round to nearest even), low half first.
__device__ __forceinline__ unsigned pack_bf16(float lo, float hi) {
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

__device__ __forceinline__ f32x4 mfma32h(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                  0, 0);
}

// Two floats to a packed f16 pair (round to nearest even), low half first.
__device__ __forceinline__ unsigned pack_f16(float lo, float hi) {
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{lo, hi}, f16x2));
}

// The f16 pair (round to nearest even) of the remainders x0 - h0, x1 - h1,
// h0 and h1 being the two halves of hw (the differences are exact in
// float32).  neg1 = -1 arrives as data: with it the compiler emits one
// mixed-precision multiply-add per value that reads the f16 half in place
// (a literal -1 turns into a subtraction after a separate conversion), and,
// unlike hand-written assembly, it sees the write and keeps the wait
// states a matrix-core read of the result needs.
__device__ __forceinline__ unsigned residual_f16(unsigned hw, float x0, float x1, float neg1) {
    const f16x2 h = __builtin_bit_cast(f16x2, hw);
    return pack_f16(fmaf((float)h[0], neg1, x0), fmaf((float)h[1], neg1, x1));
}

// Three-part bf16 split of a float32 pair into head, middle and tail words
// (low half: x0's part), each part the nearest bf16 of what the previous
// parts leave (those differences are exact in float32): |x - head| <=
// 2^-8 |x|, |x - head - middle| <= 2^-16 |x|, |x - head - middle - tail| <=
// 2^-24 |x|.  bf16 has float32's exponent range, so no part overflows or
// leaves the normal range before float32 itself would.
__device__ __forceinline__ void split3_bf16(float x0, float x1, unsigned& h, unsigned& m, unsigned& t) {
    h = pack_bf16(x0, x1);
    const float r0 = x0 - __uint_as_float(h << 16), r1 = x1 - __uint_as_float(h & 0xffff0000u);
    m = pack_bf16(r0, r1);
    const float s0 = r0 - __uint_as_float(m << 16), s1 = r1 - __uint_as_float(m & 0xffff0000u);
    t = pack_bf16(s0, s1);
}

// tanh activation of the split arithmetic: 2^11 r with r as in act_scaled,
// from (1 + 2^x) 2^-11 in one fused multiply-add (exact scaling by a power
// of two), so that the head and the remainder of 2^11 r in (0, 2048] are
// both normal f16 numbers down to r ~ 3e-8.
__device__ __forceinline__ float act_split(float x) {
    constexpr float S = 0x1p-11f;
    return __builtin_amdgcn_rcpf(fmaf(__builtin_amdgcn_exp2f(x), S, S));
}

// The float32 network's weights in registers, from the lane table (the third
// layer's stay in the table).
struct NetF32Regs {
    float A1[2][KSTEPS], A2[2][2][4];
    f32x4 B2[2];
    LaneTab lt;
    __device__ __forceinline__ explicit NetF32Regs(LaneTab table) : lt(table) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int st = 0; st < KSTEPS; ++st) A1[t][st] = lt[LT_A1 + t * KSTEPS + st];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) A2[u][t][r] = lt[LT_A2 + u * 8 + t * 4 + r];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) B2[u][r] = lt[LT_B2 + u * 4 + r];
    }
    // Layer 1 of one axis permutation for lane group q of a node tile (mrow:
    // the node's moment row, ge: the permutation's gather slots of the group).
    template <int ACT>
    __device__ __forceinline__ void layer1(const float* __restrict__ mrow, const int* __restrict__ ge,
                                           f32x4 (&Y)[8][2]) const {
        layer1_f32<act_tail(ACT)>([&](int t, int st) { return A1[t][st]; }, [&](int st) { return mrow[ge[st]]; }, Y);
    }
    template <int ACT, int DEPTH, int NS, typename Sink>
    __device__ __forceinline__ void hidden(const f32x4 (&Y)[8][2], Sink&& sink) const {
        f32x4 B2b[2] = {B2[0], B2[1]};
        if constexpr (DEPTH == 3)
#pragma unroll
            for (int v = 0; v < 2; ++v)
#pragma unroll
                for (int r = 0; r < 4; ++r) B2b[v][r] = lt[LT_B2B + v * 4 + r];
        hidden_reflections<ACT, DEPTH, NS>([&](int u, int t, int r) { return A2[u][t][r]; }, B2,
                                           [&](int v, int t, int r) { return lt[LT_A2B + v * 8 + t * 4 + r]; }, B2b, Y,
                                           []() {}, sink);
    }
};

// The group sum of a node tile and what follows it: with sums (a step
// whose adjoint follows) the sum and tilde tau into sums[node]
// [NET_SUMS_PER_NODE] (row 16 u + 4 q + r in lane (q, c)) and the rates into
// sw, else the rates into sw.
__device__ __forceinline__ void finish_tile(const f32x4 (&acc)[2], LaneTab lt, int q, int node,
                                            float* __restrict__ sw, float* __restrict__ sums) {
    if (sums) {
        float* __restrict__ row = sums + (size_t)node * NET_SUMS_PER_NODE;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) row[16 * u + 4 * q + r] = acc[u][r];
        output_layer(acc, lt, LT_W3, LT_B3, q, sw + node * 4, row + 32);
    } else {
        output_layer(acc, lt, LT_W3, LT_B3, q, sw + node * 4);
    }
}

// sums != nullptr (a step whose adjoint follows): the network values of the
// block's nodes are kept (finish_tile).
//
// DEPTH = 3: a third hidden layer (W2b, b2b) between the second layer and
// the group sum, one more product per group element whose B operand is the
// second layer's accumulator, like the second layer's is the first's.
// TPW: 16-node tiles per wavefront; wavefront w serves nodes
// [16 TPW w, 16 TPW (w + 1)) of the block.
template <int ACT, int DEPTH = 2, int TPW = 4>
__device__ __forceinline__ void network_f32(const float* __restrict__ sm, const int* __restrict__ sg,
                                            float* __restrict__ sw, LaneTab lt, int wave,
                                            int q, int c, float* __restrict__ sums = nullptr) {
    const NetF32Regs w(lt);
#pragma unroll 1
    for (int j = 0; j < TPW; ++j) {
        const int node = wave * 16 * TPW + j * 16 + c;
        const float* __restrict__ mrow = sm + node * NODE_STRIDE;
        f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll 1
        for (int p = 0; p < 6; ++p) {
            f32x4 Y[8][2];
            w.template layer1<ACT>(mrow, sg + (p * 4 + q) * GT_STRIDE, Y);
            reflections(Y);
            w.template hidden<ACT, DEPTH, 8>(Y, [&](int, const f32x4(&z)[2]) { add_act<ACT>(z, acc); });
        }
        units_in_order<ACT>(acc, q, c);
        finish_tile(acc, lt, q, node, sw, sums);
    }
}

// Small lattices: one 16-node tile per block on twelve wavefronts, three per
// SIMD: wavefront w takes half w % 2 (four reflections) of axis permutation
// w / 2, where blocks of one tile per wavefront leave most SIMDs idle and run
// the 48 group elements of a tile in series.  Each wavefront leaves the
// last-layer activations of its elements in LDS (vals [element][node]
// [hidden]); 512 threads add one (node, hidden) each in the order of the
// other block shapes, so the group sums, the rates and the step equal theirs
// bit for bit.
constexpr int PSPLIT_WAVES = 12;
constexpr int PSPLIT_ROW = 36;      // floats per (element, node) row of vals: 32 hidden, 16-byte aligned rows
constexpr int PSPLIT_VALS = 48 * 16 * PSPLIT_ROW;
constexpr int PSPLIT_FROW = 28;     // floats per node of the pulled populations, after vals in LDS
constexpr int PSPLIT_LDS = PSPLIT_VALS + 16 * PSPLIT_FROW;

template <int ACT, int DEPTH>
__device__ __forceinline__ void network_f32_psplit(const float* __restrict__ sm, const int* __restrict__ sg,
                                                   float* __restrict__ sw, LaneTab lt, int tid,
                                                   int q, int c, float* __restrict__ vals,
                                                   float* __restrict__ sums) {
    const int wave = tid >> 6;
    {
        const NetF32Regs w(lt);
        f32x4 Y[8][2];
        w.template layer1<ACT>(sm + c * NODE_STRIDE, sg + ((wave >> 1) * 4 + q) * GT_STRIDE, Y);
        reflections_half(Y, wave & 1);
        float* __restrict__ mine = vals + (wave * 4 * 16 + c) * PSPLIT_ROW + 4 * q;
        w.template hidden<ACT, DEPTH, 4>(Y, [&](int s, const f32x4(&z)[2]) {
            f32x4 h[2];
            act_f32<ACT>(z, h);
            *reinterpret_cast<f32x4*>(mine + s * 16 * PSPLIT_ROW) = h[0];
            if constexpr (act_tail(ACT) == 4) *reinterpret_cast<f32x4*>(mine + s * 16 * PSPLIT_ROW + 16) = h[1];
            if constexpr (act_tail(ACT) == 1) mine[s * 16 * PSPLIT_ROW + 16 - 3 * q] = h[1][0];
        });
    }
    __syncthreads();
    if (tid < 16 * 32 && (tid & 31) < 16 + 4 * act_tail(ACT)) {
        float* __restrict__ col = vals + (tid >> 5) * PSPLIT_ROW + (tid & 31);
        float acc = 0.0f;
#pragma unroll
        for (int g = 0; g < 48; ++g) acc += col[g * 16 * PSPLIT_ROW];
        *col = acc;
    }
    __syncthreads();
    if (wave == 0) {
        f32x4 acc[2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
            acc[u] = u && act_tail(ACT) <= q ? f32x4{0.f, 0.f, 0.f, 0.f}
                                             : *reinterpret_cast<const f32x4*>(vals + c * PSPLIT_ROW + 16 * u + 4 * q);
        finish_tile(acc, lt, q, c, sw, sums);
    }
}

// Activation feeding a split layer: 2^11 r for tanh (act_split), max(x, 0)
// for ReLU.
template <int ACT>
__device__ __forceinline__ float act_into_split(float x) {
    if constexpr (act_base(ACT) == ACT_TANH)
        return act_split(x);
    else
        return relu(x);
}

// The parts of the moment operand of one axis permutation (K slot 2 w + e
// holding x[2 w + e]): f16 head and remainder for tanh, three bf16 parts
// for ReLU.
template <int ACT>
__device__ __forceinline__ void split_input(const float (&x)[8], float neg1, u32x4 (&bp)[3]) {
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if constexpr (act_base(ACT) == ACT_TANH) {
            bp[0][w] = pack_f16(x[2 * w], x[2 * w + 1]);
            bp[1][w] = residual_f16(bp[0][w], x[2 * w], x[2 * w + 1], neg1);
            bp[2][w] = 0u;
        } else {
            unsigned h, m, t;
            split3_bf16(x[2 * w], x[2 * w + 1], h, m, t);
            bp[0][w] = h;
            bp[1][w] = m;
            bp[2][w] = t;
        }
    }
}

// The split products of one 16-row tile of A with the parts bp of B,
// accumulated from c: Ah Bh + Ah Bl + Al Bh (f16, tanh) or the six bf16
// products whose parts' orders sum to at most 2 (ReLU).
template <int ACT>
__device__ __forceinline__ f32x4 split_product(const u32x4 (&A)[3], const u32x4 (&bp)[3], f32x4 c) {
    if constexpr (act_base(ACT) == ACT_TANH) {
        c = mfma32h(A[0], bp[0], c);
        c = mfma32h(A[0], bp[1], c);
        return mfma32h(A[1], bp[0], c);
    } else {
        c = mfma32(A[0], bp[0], c);
        c = mfma32(A[0], bp[1], c);
        c = mfma32(A[1], bp[0], c);
        c = mfma32(A[0], bp[2], c);
        c = mfma32(A[2], bp[0], c);
        return mfma32(A[1], bp[1], c);
    }
}

// One split layer: the pre-activations c[u] (rows 16 u + 4 q + r, f32x4 over
// r) of A h + b for the activations h[t][r] (hidden unit 16 t + 4 q + r) of
// the previous layer, K slot 2 w + e of the products holding
// h[w / 2][2 (w % 2) + e].
//   tanh: h = 2^11 r (act_split), A = sigma W (sigma a power of two putting
//     max |A| in [128, 256)); each split into an f16 head and the f16
//     remainder, A h = Ah hh + Ah hl + Al hh (the dropped Al hl is below
//     2^-22 |A h|), three f16 products accumulated in float32 from
//     sigma 2^11 b, times back = 1 / (sigma 2^11).
//   ReLU: h unbounded, so three bf16 parts of each (split3_bf16), unscaled,
//     and the six products whose parts' orders sum to at most 2 (the dropped
//     ones are below 2^-23 |A h|), accumulated from b.
// A[u][part]: the operand parts of the layer (A[u][2] unused for tanh).
template <int ACT>
__device__ __forceinline__ void split_layer(const u32x4 (&A)[2][3], const float (&b)[2][4], float back, float neg1,
                                            const float (&h)[2][4], f32x4 (&c)[2]) {
    float x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = h[i >> 2][i & 3];
    u32x4 bp[3];
    split_input<ACT>(x, neg1, bp);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        c[u] = split_product<ACT>(A[u], bp, f32x4{b[u][0], b[u][1], b[u][2], b[u][3]});
        if constexpr (act_base(ACT) == ACT_TANH) c[u] *= back;
    }
}

// Float32-class network on the f16 / bf16 matrix cores, the products equal
// to float32's to a few units of its rounding.  tanh: every layer but the
// output one as split f16 products, layer 1 per group element like the
// bf16 network (the reflections as sign flips of the moment operand's
// parts, in Gray-code order) and scaled back by 1 / sigma_1; 12 products of
// 16x16x32 per group element and 16-node tile at depth 2.  ReLU: layer 1 on
// the float32 matrix cores with the Walsh-Hadamard fold (layer1_f32, reflections;
// split into three bf16 parts it would take 12 more products, and these
// kernels are bound by the matrix cores), the hidden-to-hidden layers as 12
// split bf16 products each.
template <int ACT, int DEPTH = 2, int TPW = 4>
__device__ __forceinline__ void network_split(const float* __restrict__ sm, const int* __restrict__ sg,
                                              float* __restrict__ sw, LaneTab lt, int wave, int q,
                                              int c) {
    auto lw = [&](int w) { return __float_as_uint(lt[w]); };
    auto lw4 = [&](int w) { return u32x4{lw(w), lw(w + 1), lw(w + 2), lw(w + 3)}; };
    constexpr int NP = act_base(ACT) == ACT_TANH ? 2 : 3;
    float B2[2][4], B3[2][4], A1[2][KSTEPS];
    u32x4 AS1[2][3], AS2[2][3], AS3[2][3], SM[3];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if constexpr (act_base(ACT) == ACT_TANH)
                AS1[u][k] = k < NP ? lw4(LS_A1 + 12 * u + 4 * k) : u32x4{0u, 0u, 0u, 0u};
            AS2[u][k] = k < NP ? lw4(LS_A2 + 12 * u + 4 * k) : u32x4{0u, 0u, 0u, 0u};
            if constexpr (DEPTH == 3) {
                AS3[u][k] = k < NP ? lw4(LS_A3 + 12 * u + 4 * k) : u32x4{0u, 0u, 0u, 0u};
            }
        }
    if constexpr (act_base(ACT) == ACT_TANH) {
#pragma unroll
        for (int b = 0; b < 3; ++b)
            SM[b] = lw4(LS_SM + 4 * b);
    } else {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int st = 0; st < KSTEPS; ++st) A1[t][st] = lt[LT_A1 + t * KSTEPS + st];
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            B2[u][r] = lt[LS_B2 + u * 4 + r];
            B3[u][r] = DEPTH == 3 ? lt[LS_B3 + u * 4 + r] : 0.0f;
        }
    const float back1 = lt[LS_BACK], back2 = lt[LS_BACK + 1], back3 = lt[LS_BACK + 2], neg1 = lt[LS_NEG1];

#pragma unroll 1
    for (int j = 0; j < TPW; ++j) {
        const int node = wave * 16 * TPW + j * 16 + c;
        const float* __restrict__ mrow = sm + node * NODE_STRIDE;
        f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll 1
        for (int p = 0; p < 6; ++p) {
            const int* __restrict__ ge = sg + (p * 4 + q) * GT_STRIDE;
            u32x4 bp[3];
            f32x4 Y[8][2];
            if constexpr (act_base(ACT) == ACT_TANH) {
                float x[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = mrow[ge[i]];
                split_input<ACT>(x, neg1, bp);
            } else {
                layer1_f32([&](int t, int st) { return A1[t][st]; }, [&](int st) { return mrow[ge[st]]; }, Y);
                reflections(Y);
            }
            // tanh: the 8 reflections in Gray-code order, consecutive ones
            // differing in one reflection bit: one mask XOR per word and part.
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                float h1[2][4];
                if constexpr (act_base(ACT) == ACT_TANH) {
                    if (k > 0)
#pragma unroll
                        for (int e = 0; e < NP; ++e) bp[e] ^= SM[__builtin_ctz(k)];
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const f32x4 c1 = split_product<ACT>(AS1[t], bp, f32x4{0.f, 0.f, 0.f, 0.f}) * back1;
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            h1[t][r] = r < act_values(ACT, t) ? act_into_split<ACT>(c1[r]) : 0.0f;
                    }
                } else {
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            h1[t][r] = r < act_values(ACT, t) ? act_into_split<ACT>(Y[k][t][r]) : 0.0f;
                }
                f32x4 cz[2];
                split_layer<ACT>(AS2, B2, back2, neg1, h1, cz);
                if constexpr (DEPTH == 3) {
                    float h2[2][4];
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            h2[u][r] = r < act_values(ACT, u) ? act_into_split<ACT>(cz[u][r]) : 0.0f;
                    split_layer<ACT>(AS3, B3, back3, neg1, h2, cz);
                }
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int r = 0; r < act_values(ACT, u); ++r) acc[u][r] += act_scaled<ACT>(cz[u][r]);
            }
        }
        units_in_order<ACT>(acc, q, c);
        output_layer(acc, lt, LS_W3, LS_B3O, q, sw + node * 4);
    }
}

// DEPTH 3: the third hidden layer as one more bf16 product per group
// element, fed by the second layer's activations packed like the first's.
template <int ACT, int DEPTH = 2, int TPW = 4>
__device__ __forceinline__ void network_bf16(const float* __restrict__ sm, const int* __restrict__ sg,
                                             float* __restrict__ sw, LaneTab lt, int wave,
                                             int q, int c) {
    auto lw = [&](int w) { return __float_as_uint(lt[w]); };
    auto lw4 = [&](int w) { return u32x4{lw(w), lw(w + 1), lw(w + 2), lw(w + 3)}; };
    u32x4 A1[2], A2[2], SM[3], A3[2];
    float B2[2][4], B3[2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t)
        A1[t] = lw4(LB_A1 + 4 * t);
#pragma unroll
    for (int u = 0; u < 2; ++u)
        A2[u] = lw4(LB_A2 + 4 * u);
#pragma unroll
    for (int b = 0; b < 3; ++b)
        SM[b] = lw4(LB_SM + 4 * b);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) B2[u][r] = lt[LB_B2 + u * 4 + r];
    if constexpr (DEPTH == 3) {
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            A3[v] = lw4(LB_A2B + 4 * v);
#pragma unroll
            for (int r = 0; r < 4; ++r) B3[v][r] = lt[LB_B2B + v * 4 + r];
        }
    }

#pragma unroll 1
    for (int j = 0; j < TPW; ++j) {
        const int node = wave * 16 * TPW + j * 16 + c;
        const float* __restrict__ mrow = sm + node * NODE_STRIDE;
        f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll 1
        for (int p = 0; p < 6; ++p) {
            const int* __restrict__ ge = sg + (p * 4 + q) * GT_STRIDE;
            float x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = mrow[ge[i]];
            const u32x4 xb = {pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]), pack_bf16(x[4], x[5]),
                              pack_bf16(x[6], x[7])};
            // The 8 reflections in Gray-code order k ^ (k >> 1): consecutive
            // ones differ in one reflection bit (bit ctz(k)), so one mask XOR
            // per word moves to the next instead of one per set bit.
            u32x4 bs = xb;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (k > 0) bs ^= SM[__builtin_ctz(k)];
                f32x4 c1[2];
#pragma unroll
                for (int t = 0; t < 2; ++t) c1[t] = mfma32(A1[t], bs, f32x4{0.f, 0.f, 0.f, 0.f});
                float h[2][4];
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) h[t][r] = r < act_values(ACT, t) ? act_scaled<ACT>(c1[t][r]) : 0.0f;
                const u32x4 hb = {pack_bf16(h[0][0], h[0][1]), pack_bf16(h[0][2], h[0][3]),
                                  pack_bf16(h[1][0], h[1][1]), pack_bf16(h[1][2], h[1][3])};
                f32x4 c2[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) c2[u] = mfma32(A2[u], hb, f32x4{B2[u][0], B2[u][1], B2[u][2], B2[u][3]});
                if constexpr (DEPTH == 3) {
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int r = 0; r < 4; ++r) h[u][r] = r < act_values(ACT, u) ? act_scaled<ACT>(c2[u][r]) : 0.0f;
                    const u32x4 h2b = {pack_bf16(h[0][0], h[0][1]), pack_bf16(h[0][2], h[0][3]),
                                       pack_bf16(h[1][0], h[1][1]), pack_bf16(h[1][2], h[1][3])};
#pragma unroll
                    for (int v = 0; v < 2; ++v)
                        c2[v] = mfma32(A3[v], h2b, f32x4{B3[v][0], B3[v][1], B3[v][2], B3[v][3]});
                }
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int r = 0; r < act_values(ACT, u); ++r) acc[u][r] += act_scaled<ACT>(c2[u][r]);
            }
        }
        units_in_order<ACT>(acc, q, c);
        output_layer(acc, lt, LB_W3, LB_B3, q, sw + node * 4);
    }
}

// RATES = true: no streaming, the rates of the stored state are written to
// omega_out [4][n] instead of a step (readout and tests of the network alone).
// Work space of one block in LDS, declared by each kernel.  A block serves
// NODES = 256 or 64 nodes with TPW 16-node tiles per wavefront, so
// 64 NODES / (16 TPW) threads: 256 nodes on 4 wavefronts (TPW 4), 64 nodes on
// one wavefront (TPW 4) or on 4 wavefronts of one tile each (TPW 1, the
// shortest serial chain per wavefront, for small lattices).  The wavefronts
// of a block share only the gather table; every variant does the same
// arithmetic per node.
struct BlockLds {
    float* sm;      // [NODES][NODE_STRIDE] moments, then hidden activations
    int* sg;        // [GT_ENTRIES] gather table
    float* sw;      // [NODES][4] rates
    float* vals = nullptr;  // [PSPLIT_LDS] activations and populations (twelve-wavefront tiles)
};

template <int S, int ACT, bool RATES, int PREC, int NODES, int DEPTH = 2, int TPW = 4, bool SUMS = false>
__device__ __forceinline__ void nco_mfma_block(const typename Codec<S>::store_t* __restrict__ fin,
                                               typename Codec<S>::store_t* __restrict__ fout, const StepArgs& a,
                                               const float* __restrict__ lane_tab, const int* __restrict__ gtab,
                                               double* __restrict__ omega_out, int blk, BlockLds lds);

#define NCO_BLOCK_LDS(NODES)                         \
    __shared__ float lds_sm[(NODES) * NODE_STRIDE];  \
    __shared__ int lds_sg[GT_ENTRIES];               \
    __shared__ float lds_sw[(NODES) * 4];            \
    const BlockLds lds{lds_sm, lds_sg, lds_sw};

// TPW = 0: the twelve-wavefront tile of network_f32_psplit (16 nodes).
constexpr int mfma_block_threads(int nodes, int tpw) { return tpw == 0 ? PSPLIT_WAVES * 64 : nodes / (16 * tpw) * 64; }

// Waves per SIMD the register allocation must leave room for: 3 for the
// split networks (156 VGPRs for tanh at depth 2; the others spill 12-57
// registers into scratch and still run 1-7 % faster than at 2 waves, the
// third wave keeping their vector instructions issuing) and for the float32
// steps (151-169 VGPRs unconstrained at depth 2, 177 at depth 3; at 168, 0-17
// spilled, depth 3 4 % faster at 128^3 and 8 % on a 16^3 lattice) - but for
// depth 2 with one tile per wavefront, where the lattice has no third wave to
// offer a SIMD and the constraint only costs (24^3 30.2 against 32.7 us, 32^3
// 53.5 against 57.8) -, 4 for float32 networks of at most 20 units (0-4 spilled;
// depth 3, ReLU: 24^3 28.6 -> 25.9 us, 96^3 1.035 -> 1.022 ms) and for the bf16
// depth-3 steps (ReLU 132 VGPRs unconstrained, 128 without spills at 4 waves,
// 2 % faster), no constraint otherwise.
constexpr int mfma_min_waves(int act, int prec, int depth, int tpw, bool sums) {
    return prec == MLP_PREC_BF16 && depth == 3 ? 4
           : prec == MLP_PREC_F32 && sums && act_tail(act) < 4 && tpw != 0 ? 4
           : prec == MLP_PREC_F32S || (prec == MLP_PREC_F32 && sums && (depth == 3 || tpw != 1)) ? 3
                                                                                                   : 1;
}

template <int S, int ACT, bool RATES, int PREC, int NODES, int DEPTH, int TPW, bool SUMS = false>
__global__ __launch_bounds__(mfma_block_threads(NODES, TPW))
__attribute__((amdgpu_waves_per_eu(mfma_min_waves(ACT, PREC, DEPTH, TPW, SUMS)))) void k_nco_mfma(
    const typename Codec<S>::store_t* __restrict__ fin, typename Codec<S>::store_t* __restrict__ fout,
    StepArgs a, const float* __restrict__ lane_tab, const int* __restrict__ gtab, double* __restrict__ omega_out) {
    NCO_BLOCK_LDS(NODES)
    if constexpr (TPW == 0) {
        __shared__ __align__(16) float lds_vals[PSPLIT_LDS];
        BlockLds lv = lds;
        lv.vals = lds_vals;
        nco_mfma_block<S, ACT, RATES, PREC, NODES, DEPTH, TPW, SUMS>(fin, fout, a, lane_tab, gtab, omega_out,
                                                               xcd_block(blockIdx.x, gridDim.x), lv);
    } else {
        nco_mfma_block<S, ACT, RATES, PREC, NODES, DEPTH, TPW, SUMS>(fin, fout, a, lane_tab, gtab, omega_out,
                                                               xcd_block(blockIdx.x, gridDim.x), lds);
    }
}

template <int S, int ACT, int PREC>
__device__ __forceinline__ void grouped_block(const GroupDesc& d, int blk, BlockLds lds) {
    using T = typename Codec<S>::store_t;
    // The float32 network through the instantiation with the (here unused)
    // network-value branch, for its register allocation (see
    // launch_kind).
    nco_mfma_block<S, ACT, false, PREC, 256, 2, 4, PREC == MLP_PREC_F32>(
        static_cast<const T*>(d.fin), static_cast<T*>(d.fout), d.a, d.lane_tab, d.gtab, nullptr, blk, lds);
}

// One step of several lattices with the same storage, activation and
// network arithmetic.
template <int S, int ACT, int PREC>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(PREC == MLP_PREC_F32 ? 3 : 1))) void k_nco_mfma_grouped(LaunchGroup g) {
    NCO_BLOCK_LDS(256)
    const int i = group_member(g, blockIdx.x);
    grouped_block<S, ACT, PREC>(g.d[i], blockIdx.x - g.prefix[i], lds);
}

template <int S, int ACT, bool RATES, int PREC, int NODES, int DEPTH, int TPW, bool SUMS>
__device__ __forceinline__ void nco_mfma_block(const typename Codec<S>::store_t* __restrict__ fin,
                                               typename Codec<S>::store_t* __restrict__ fout, const StepArgs& a,
                                               const float* __restrict__ lane_tab, const int* __restrict__ gtab,
                                               double* __restrict__ omega_out, int blk, BlockLds lds) {
    constexpr int THREADS = mfma_block_threads(NODES, TPW);
    float* __restrict__ sm = lds.sm;
    int* __restrict__ sg = lds.sg;
    float* __restrict__ sw = lds.sw;
    const int tid = threadIdx.x;
    const int idx = blk * NODES + tid;
    const bool live = (THREADS == NODES || tid < NODES) && idx < a.n;

    for (int e = tid; e < GT_ENTRIES; e += THREADS) sg[e] = gtab[e];

    // Phase A: pull and transform to moments.
    if constexpr (TPW == 0) {
        // Twelve-wavefront tiles: the tile's 16 x 27 pulls spread over the
        // block's threads (each a load or a folded one at the faces of the
        // reduced cube), kept in LDS for the relaxation as well.
        static_assert(!RATES, "twelve-wavefront tiles run steps");
        float* __restrict__ fl = lds.vals + PSPLIT_VALS;
        for (int e = tid; e < NODES * Q; e += THREADS) {
            const int nd = e % NODES, i = e / NODES, id = blk * NODES + nd;
            fl[nd * PSPLIT_FROW + i] =
                id < a.n ? pull_one<S>(fin, a, node_of(id, a.nx, a.ny), i) : (float)weight_of(i);
        }
        __syncthreads();
        if (tid < NODES) {
            float f[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i) f[i] = fl[tid * PSPLIT_FROW + i];
            float m[Q];
            to_moments(f, m);
            float* row = sm + tid * NODE_STRIDE;
#pragma unroll
            for (int k = 0; k < Q; ++k) row[k] = m[row_tensor(k)];
            row[27] = 1.0f;
            row[28] = 0.0f;
        }
    } else if (THREADS == NODES || tid < NODES) {
        float f[Q];
        if (live) {
            if constexpr (RATES)
                load_local<S>(fin, a.n, idx, f);
            else
                pull<S>(fin, a, node_of(idx, a.nx, a.ny), f);
        } else {
#pragma unroll
            for (int i = 0; i < Q; ++i) f[i] = (float)weight_of(i);
        }
        float m[Q];
        to_moments(f, m);
        float* row = sm + tid * NODE_STRIDE;
#pragma unroll
        for (int k = 0; k < Q; ++k) row[k] = m[row_tensor(k)];
        row[27] = 1.0f;
        row[28] = 0.0f;
    }
    __syncthreads();

    // Phase B: the network, one wavefront per 64 nodes.
    {
        const int lane = tid & 63;
        const LaneTab lt(lane_tab, lane);
        if constexpr (TPW == 0) {
            static_assert(PREC == MLP_PREC_F32 && NODES == 16, "twelve-wavefront tiles: the float32 network");
            float* sums = SUMS && a.net_sums ? a.net_sums + (size_t)blk * NODES * NET_SUMS_PER_NODE : nullptr;
            network_f32_psplit<ACT, DEPTH>(sm, sg, sw, lt, tid, lane >> 4, lane & 15, lds.vals, sums);
        } else if constexpr (PREC == MLP_PREC_BF16) {
            network_bf16<ACT, DEPTH, TPW>(sm, sg, sw, lt, tid >> 6, lane >> 4, lane & 15);
        } else if constexpr (PREC == MLP_PREC_F32S) {
            static_assert(!SUMS, "the split arithmetic keeps no network values");
            network_split<ACT, DEPTH, TPW>(sm, sg, sw, lt, tid >> 6, lane >> 4, lane & 15);
        } else if constexpr (SUMS) {
            // Keeps the network values when a.net_sums is set, else a plain
            // step (a uniform branch after each tile).
            float* sums = a.net_sums ? a.net_sums + (size_t)blk * NODES * NET_SUMS_PER_NODE : nullptr;
            network_f32<ACT, DEPTH, TPW>(sm, sg, sw, lt, tid >> 6, lane >> 4, lane & 15, sums);
        } else {
            network_f32<ACT, DEPTH, TPW>(sm, sg, sw, lt, tid >> 6, lane >> 4, lane & 15);
        }
    }
    __syncthreads();

    if constexpr (RATES) {
        if (live)
#pragma unroll
            for (int n = 0; n < 4; ++n) omega_out[(size_t)n * a.n + idx] = (double)sw[tid * 4 + n];
        return;
    }

    // Phase C: relax with the rates and store.
    if (live) {
        float f[Q], m[Q];
        if constexpr (TPW == 0) {
#pragma unroll
            for (int i = 0; i < Q; ++i) f[i] = lds.vals[PSPLIT_VALS + tid * PSPLIT_FROW + i];
        } else {
            pull<S>(fin, a, node_of(idx, a.nx, a.ny), f);
        }
        const float* row = sm + tid * NODE_STRIDE;
#pragma unroll
        for (int k = 0; k < Q; ++k) m[row_tensor(k)] = row[k];
        float omega[4];
#pragma unroll
        for (int n = 0; n < 4; ++n) omega[n] = sw[tid * 4 + n];
        float dm[Q], df[Q];
        if (a.n_modes > 0) {
            float Fx, Fy, Fz;
            read_force(a, idx, Fx, Fy, Fz);
            collision_delta<float, true>(m, a.omega_nu_f, omega, Fx, Fy, Fz, dm);
        } else {
            collision_delta<float, false>(m, a.omega_nu_f, omega, 0.f, 0.f, 0.f, dm);
        }
        from_moments(dm, df);
#pragma unroll
        for (int i = 0; i < Q; ++i) f[i] -= df[i];
        store_local<S>(fout, a.n, idx, f, a.sr_key);
    }
}

// Block shape of the single-lattice kernel (the results are bit-identical
// for all three).  About 2 wavefronts per SIMD are resident (8 per CU).
// Below 65536 nodes, 64-node blocks with one tile per wavefront finish in
// fewer rounds of tiles (4x fewer up to 32768 nodes).  Up to 131072 nodes,
// one-wavefront 64-node blocks (measured 10 % faster than 256-node blocks at
// 32^3 before the one-tile blocks existed, equal from 64^3 up).  Above, the
// 256-node blocks.
enum MfmaBlock { MFMA_BLOCK_256 = 0, MFMA_BLOCK_64 = 1, MFMA_BLOCK_64_TILE = 2 };
// Float32-network steps of lattices up to this many nodes run twelve-wavefront
// tiles (network_f32_psplit): 256 blocks, one round over the 256 CUs.  A
// block holds 111 KB of LDS, one per CU, so beyond that the blocks run in
// rounds and the one-tile-per-wavefront blocks are faster (16^3: 12.6 against
// 30 us per step; in six-wavefront tiles of the same rounds, 24^3: 53 against 31).
constexpr int PSPLIT_MAX_NODES = 4096;
constexpr int mfma_block_kind(int n) {
    return n < 65536 ? MFMA_BLOCK_64_TILE : n < 2 * 256 * 256 ? MFMA_BLOCK_64 : MFMA_BLOCK_256;
}

// A step, or with omega_out the rates of the state (one shape).
template <int S, int ACT, int PP, int DD>
hipError_t launch_kind(const void* fin_, void* fout_, const StepArgs& a, const float* lane_tab, const int* gtab,
                       double* omega_out, hipStream_t st) {
    using T = typename Codec<S>::store_t;
    const T* fin = static_cast<const T*>(fin_);
    T* fout = static_cast<T*>(fout_);
    // Float32 networks: the instantiation that can keep the network values
    // for the adjoint (when a.net_sums is set) runs the plain steps too: with
    // that branch the compiler allocates 154-161 VGPRs at depth 2, 3 waves
    // per SIMD, where the instantiation without it takes 230 and 2 waves and
    // runs 3 % slower; at depth 3, 177 against 254 (with mfma_min_waves, 3
    // waves).
    constexpr bool SUMS = PP == MLP_PREC_F32;
    if (!SUMS && a.net_sums) return hipErrorInvalidValue;
    const int kind = mfma_block_kind(a.n);
#define NCO_LAUNCH(RATES, NODES, TPW, KEEP)                                                                       \
    hipLaunchKernelGGL((k_nco_mfma<S, ACT, RATES, PP, NODES, DD, TPW, KEEP>), dim3((a.n + NODES - 1) / NODES),     \
                       dim3(mfma_block_threads(NODES, TPW)), 0, st, fin, fout, a, lane_tab, gtab, omega_out)
    if (omega_out) {
        NCO_LAUNCH(true, 64, 1, false);
        return hipGetLastError();
    }
    if constexpr (PP == MLP_PREC_F32)
        if (a.n <= PSPLIT_MAX_NODES) {
            NCO_LAUNCH(false, 16, 0, true);
            return hipGetLastError();
        }
    // 256-node blocks: not for the unfolded float32 network, whose smaller
    // ones tie with them at every size.
    constexpr bool FULL = act_base(ACT) == ACT_TANH_FULL || act_tail(ACT) == 0;
    if (kind == MFMA_BLOCK_64_TILE)
        NCO_LAUNCH(false, 64, 1, SUMS);
    else if (FULL || kind == MFMA_BLOCK_64)
        NCO_LAUNCH(false, 64, 4, SUMS);
    else if constexpr (!FULL)
        NCO_LAUNCH(false, 256, 4, SUMS);
#undef NCO_LAUNCH
    return hipGetLastError();
}

// The form of a network of `units` hidden units (act_tail): five of eight
// values per lane up to 20 (width 20, ReLU, 128^3: float32 2.15 -> 1.43 ms, bf16
// 0.602 -> 0.475, split 1.50 -> 1.25; depth 3 float32 3.65 -> 2.39; 16^3 12.6 ->
// 9.8 us).
template <int S, int BASE, int PP>
hipError_t launch_units(const void* fin, void* fout, const StepArgs& a, const float* lane_tab, const int* gtab,
                        double* omega_out, hipStream_t st) {
    if (a.depth == 3)
        return a.units <= 20 ? launch_kind<S, BASE + UNITS_20, PP, 3>(fin, fout, a, lane_tab, gtab, omega_out, st)
                             : launch_kind<S, BASE, PP, 3>(fin, fout, a, lane_tab, gtab, omega_out, st);
    return a.units <= 20 ? launch_kind<S, BASE + UNITS_20, PP, 2>(fin, fout, a, lane_tab, gtab, omega_out, st)
                         : launch_kind<S, BASE, PP, 2>(fin, fout, a, lane_tab, gtab, omega_out, st);
}

template <int PP>
hipError_t launch_prec(int storage, const void* fin, void* fout, const StepArgs& a, const float* lane_tab,
                       const int* gtab, double* omega_out, hipStream_t st) {
#define NCO_STORAGE(SS)                                                                                          \
    case SS:                                                                                                     \
        return a.act == ACT_TANH ? launch_units<SS, ACT_TANH, PP>(fin, fout, a, lane_tab, gtab, omega_out, st)   \
                                 : launch_units<SS, ACT_RELU, PP>(fin, fout, a, lane_tab, gtab, omega_out, st);
    switch (storage) {
        NCO_STORAGE(ST_F32)
        NCO_STORAGE(ST_F16)
        NCO_STORAGE(ST_BF16)
        default: return hipErrorInvalidValue;
    }
#undef NCO_STORAGE
}

template <int PP>
hipError_t launch_prec_grouped(int storage, int act, int units, const LaunchGroup& g, hipStream_t st) {
    const dim3 grid(g.prefix[g.count]), block(256);
#define NCO_GROUP(SS, AA)                                                                                  \
    if (units <= 20)                                                                                       \
        hipLaunchKernelGGL((k_nco_mfma_grouped<SS, AA + UNITS_20, PP>), grid, block, 0, st, g);            \
    else                                                                                                   \
        hipLaunchKernelGGL((k_nco_mfma_grouped<SS, AA, PP>), grid, block, 0, st, g);
#define NCO_STORAGE(SS)             \
    case SS:                        \
        if (act == ACT_TANH) {      \
            NCO_GROUP(SS, ACT_TANH) \
        } else {                    \
            NCO_GROUP(SS, ACT_RELU) \
        }                           \
        return hipGetLastError();
    switch (storage) {
        NCO_STORAGE(ST_F32)
        NCO_STORAGE(ST_F16)
        NCO_STORAGE(ST_BF16)
        default: return hipErrorInvalidValue;
    }
#undef NCO_STORAGE
#undef NCO_GROUP
}

}  // namespace

// One step fin -> fout, or with omega_out the rates of the state in fin, of
// each arithmetic.
#define NCO_NET_DECL(NAME)                                                                                       \
    hipError_t launch_net_##NAME(int storage, const void* fin, void* fout, const StepArgs& a, const float* lane_tab, \
                                 const int* gtab, double* omega_out, hipStream_t st);                            \
    hipError_t launch_net_##NAME##_grouped(int storage, int act, int units, const LaunchGroup& g, hipStream_t st);
NCO_NET_DECL(f32)
NCO_NET_DECL(split)
NCO_NET_DECL(bf16)
#undef NCO_NET_DECL
hipError_t launch_net_full(int storage, const void* fin, void* fout, const StepArgs& a, const float* lane_tab,
                           const int* gtab, double* omega_out, hipStream_t st);

// The two functions of one arithmetic.
#define NCO_NET_DEFINE(NAME, PP)                                                                                 \
    hipError_t launch_net_##NAME(int storage, const void* fin, void* fout, const StepArgs& a, const float* lane_tab, \
                                 const int* gtab, double* omega_out, hipStream_t st) {                           \
        return launch_prec<PP>(storage, fin, fout, a, lane_tab, gtab, omega_out, st);                            \
    }                                                                                                            \
    hipError_t launch_net_##NAME##_grouped(int storage, int act, int units, const LaunchGroup& g, hipStream_t st) { \
        return launch_prec_grouped<PP>(storage, act, units, g, st);                                              \
    }

}  // namespace nco
