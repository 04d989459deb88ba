// The float32 matrix-core network's device pieces, shared by the forward
// step (nco_mfma.hip) and the reverse step (nco_adjoint.hip): both run the
// same products in the same order, so the reverse step's own forward pass
// gives the values the forward step keeps, bit for bit.
#pragma once

#include "fold.h"
#include "kernels.h"

namespace nco {

constexpr int MW = 32;              // network width on the matrix-core paths

typedef float f32x4 __attribute__((ext_vector_type(4)));

// The per-lane table of a matrix-core network: LANE_WORDS 4-byte words per
// lane, in one run.  (Quads of words interleaved over the lanes, so that a
// wavefront's loads are contiguous, gave 1-2 % on the depth-2 networks and
// cost 1-7 % on the others: the loads are short and cached, and the four-word
// register tuples they arrive in raise the register count.)
constexpr int LANE_WORDS = 144;

template <typename T>
struct LaneTabT {
    T* p;
    __host__ __device__ LaneTabT(T* table, int lane) : p(table + LANE_WORDS * lane) {}
    __host__ __device__ __forceinline__ T& operator[](int w) const { return p[w]; }
};
using LaneTab = LaneTabT<const float>;

// Offsets in the per-lane table of the float32 network.
constexpr int LT_A1 = 0;            // [t 2][st 10]    W1 rows / b1 as A operand
constexpr int LT_A2 = 20;           // [u 2][t 2][r 4] W2 as A operand
constexpr int LT_B2 = 36;           // [u 2][r 4]      b2 as accumulator init
constexpr int LT_W3 = 44;           // [u 2][r 4][n 4] W3 / 48
constexpr int LT_B3 = 76;           // [n 4]
constexpr int LT_A2B = 80;          // [v 2][t 2][r 4] W2b as A operand (depth 3)
constexpr int LT_B2B = 96;          // [v 2][r 4]      b2b as accumulator init (depth 3)

// Hidden units of a layer lie in two 16-row tiles; a lane (q, c) holds rows
// 4 q .. 4 q + 3 of each.  Tile 0 is units 0 .. 15 in order.  Tile 1 is units
// 16 .. 31 in order (tail 4), or, in networks of at most 20 units, unit 16 + j
// in row 4 j and nothing else (UNITS_20, tail 1), so that every lane holds one
// of them in its first register: five activations per lane and layer instead
// of eight, and five K-steps of a float32 product instead of eight (the
// products of the other rows would add exact zeros).  UNITS_16 (tail 0) leaves
// tile 1 out.
constexpr int act_base(int act) { return act & 7; }
constexpr int act_tail(int act) { return act & UNITS_16 ? 0 : act & UNITS_20 ? 1 : 4; }
constexpr int act_values(int act, int t) { return t == 0 ? 4 : act_tail(act); }
// The unit in row 4 q + r of tile t, -1 for none.
constexpr int tile_unit(bool units20, int t, int q, int r) {
    return t == 0 ? 4 * q + r : !units20 ? 16 + 4 * q + r : r == 0 ? 16 + q : -1;
}

// A group sum in the order of tail 4, from lanes in the order of ACT.
template <int ACT>
__device__ __forceinline__ void units_in_order(f32x4 (&acc)[2], int q, int c) {
    if constexpr (act_tail(ACT) == 1) {
        const float v = acc[1][0];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float w = __shfl(v, 16 * r + c, 64);
            acc[1][r] = q == 0 ? w : 0.0f;
        }
    }
}

// max(x, 0), 0 for a NaN, as the median of x, 0 and infinity: one instruction,
// where fmaxf takes two on a product's result (the first quiets it, in case it
// were a signalling NaN; the median of a visible infinity becomes that fmaxf).
// Width 20, 128^3, steps in a long run: bf16 0.475 -> 0.406 ms, depth 3 0.664 ->
// 0.525, float32 1.43 -> 1.38.
__device__ __forceinline__ float relu(float x) {
    float inf = __builtin_inff();
    asm("" : "+s"(inf));
    return __builtin_amdgcn_fmed3f(x, 0.0f, inf);
}

// Activation as evaluated on the matrix-core paths.  For tanh the
// pre-activation arrives scaled by kappa = 2 log2(e) and the function returns
// r = 1 / (1 + 2^(kappa z)), so that tanh(z) = 1 - 2 r; the affine map 1 - 2 r
// is folded into the next layer's weights and bias on the host (and into W3,
// b3 for the group sum), which leaves exp2, add and reciprocal per value.  r
// saturates correctly (2^+inf = inf gives 0).
//
// ACT_TANH_FULL (the float32 network that is not folded): tanh within 1.3
// units of the last place plus the hardware exp2's and reciprocal's, against
// the folded form's absolute 1e-7.  |x| < 0.9: x + x s P(s), s = x^2, P the
// degree-5 least-maximum fit of (tanh(x) / x - 1) / s (1.6e-8 relative);
// above, 1 - 2 / (1 + e^(2 |x|)) with x's sign.  Both sides are evaluated:
// 22 issue slots, two of the instructions at quarter rate.
template <int ACT>
__device__ __forceinline__ float act_scaled(float x) {
    if constexpr (act_base(ACT) == ACT_RELU) {
        return relu(x);
    } else if constexpr (act_base(ACT) == ACT_TANH_FULL) {
        const float a = fabsf(x), s = x * x;
        float p = fmaf(1.30395428e-3f, s, -6.86004246e-3f);
        p = fmaf(p, s, 2.09041145e-2f);
        p = fmaf(p, s, -5.37214838e-2f);
        p = fmaf(p, s, 1.33303598e-1f);
        p = fmaf(p, s, -3.33332121e-1f);
        const float e = __builtin_amdgcn_exp2f(a * (float)(2.0 / 0.69314718055994530942));
        const float big = copysignf(fmaf(-2.0f, __builtin_amdgcn_rcpf(1.0f + e), 1.0f), x);
        return a < 0.9f ? fmaf(p * s, x, x) : big;
    } else {
        return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(x));
    }
}

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// The eight parity-class partial products of layer 1 of one axis permutation
// over 10 K-steps (A1(t, st): W1's A operand, b(st): the moment operand), and
// their Walsh-Hadamard transform over the class index, after which Y[s][t] is
// the pre-activation of reflection pattern s (hidden rows 16 t + 4 q + r).
// TAIL as act_tail (0: Y[.][1] = 0).
template <int TAIL = 4, typename A, typename B>
__device__ __forceinline__ void layer1_f32(A&& A1, B&& b, f32x4 (&Y)[8][2]) {
    // Moment operand of this permutation, one K-step per register.
    float x[KSTEPS];
#pragma unroll
    for (int st = 0; st < KSTEPS; ++st) x[st] = b(st);
#pragma unroll
    for (int ci = 0; ci < 8; ++ci) {
        Y[ci][0] = f32x4{0.f, 0.f, 0.f, 0.f};
        Y[ci][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int st = 0; st < KSTEPS; ++st)
#pragma unroll
        for (int t = 0; t < (TAIL ? 2 : 1); ++t) Y[step_class(st)][t] = mfma4(A1(t, st), x[st], Y[step_class(st)][t]);
}

__device__ __forceinline__ void reflections(f32x4 (&Y)[8][2]) {
#pragma unroll
    for (int bit = 1; bit < 8; bit <<= 1)
#pragma unroll
        for (int ci = 0; ci < 8; ++ci)
            if (!(ci & bit))
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const f32x4 u0 = Y[ci][t], u1 = Y[ci | bit][t];
                    Y[ci][t] = u0 + u1;
                    Y[ci | bit][t] = u0 - u1;
                }
}

// The reflections 4 half .. 4 half + 3 only (their transform's last level
// keeps one side), into Y[0 .. 3].
__device__ __forceinline__ void reflections_half(f32x4 (&Y)[8][2], int half) {
#pragma unroll
    for (int bit = 1; bit < 4; bit <<= 1)
#pragma unroll
        for (int ci = 0; ci < 8; ++ci)
            if (!(ci & bit))
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const f32x4 u0 = Y[ci][t], u1 = Y[ci | bit][t];
                    Y[ci][t] = u0 + u1;
                    Y[ci | bit][t] = u0 - u1;
                }
    const float sign = half ? -1.0f : 1.0f;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) Y[s][t][r] = fmaf(sign, Y[4 + s][t][r], Y[s][t][r]);
}

// One hidden-to-hidden layer, c[u] += A(u, t, r) h[t][r] over its K-steps.
template <int TAIL = 4, typename A>
__device__ __forceinline__ void hidden_f32(A&& A2, const f32x4 (&h)[2], f32x4 (&c)[2]) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < (t == 0 ? 4 : TAIL); ++r)
#pragma unroll
            for (int u = 0; u < (TAIL ? 2 : 1); ++u) c[u] = mfma4(A2(u, t, r), h[t][r], c[u]);
}

template <int ACT>
__device__ __forceinline__ void act_f32(const f32x4 (&z)[2], f32x4 (&h)[2]) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) h[t][r] = r < act_values(ACT, t) ? act_scaled<ACT>(z[t][r]) : 0.0f;
}

// Hides a lane's place in a weight table from the compiler, so that weights
// read through it from here on are read where they are used instead of being
// kept in registers for the whole reflection loop.
__device__ __forceinline__ void fresh_lane(int& place) { asm("" : "+v"(place)); }

// Reflections 0 .. NS - 1 (pre-activations Y) through the hidden layers; the
// last layer's pre-activations of reflection s go to sink(s, z), in order.
//
// Depth 2 is software-pipelined over the reflections: while the 16 products
// of reflection s run on the matrix cores, the vector units activate layer 1
// of reflection s + 1 and layer 2 of reflection s - 1 (independent of them).
// fresh() runs before each reflection (see fresh_lane).
template <int ACT, int DEPTH, int NS, typename A, typename AB, typename Fresh, typename Sink>
__device__ __forceinline__ void hidden_reflections(A&& A2, const f32x4 (&B2)[2], AB&& A2b, const f32x4 (&B2b)[2],
                                                   const f32x4 (&Y)[8][2], Fresh&& fresh, Sink&& sink) {
    if constexpr (DEPTH == 3) {
        // Unrolled: Y[s] must stay in registers.
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            f32x4 h[2], c[2] = {B2[0], B2[1]}, c3[2] = {B2b[0], B2b[1]};
            fresh();
            act_f32<ACT>(Y[s], h);
            hidden_f32<act_tail(ACT)>(A2, h, c);
            act_f32<ACT>(c, h);
            hidden_f32<act_tail(ACT)>(A2b, h, c3);
            sink(s, c3);
        }
        return;
    }
    f32x4 h[2], prev[2];
    act_f32<ACT>(Y[0], h);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        f32x4 c[2] = {B2[0], B2[1]};
        hidden_f32<act_tail(ACT)>(A2, h, c);
        if (s > 0) sink(s - 1, prev);
        if (s < NS - 1) act_f32<ACT>(Y[s + 1], h);
        prev[0] = c[0];
        prev[1] = c[1];
    }
    sink(NS - 1, prev);
}

// The group sum adds the last layer's activations element by element, in the
// order (permutation, reflection), in every block shape.
template <int ACT>
__device__ __forceinline__ void add_act(const f32x4 (&z)[2], f32x4 (&acc)[2]) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < act_values(ACT, u); ++r) acc[u][r] += act_scaled<ACT>(z[u][r]);
}

// Output layer on the group sum of one node tile and the rate squashing;
// w3 and b3 are the layer's offsets in the lane's table; the lanes of group
// q = 0 write the four rates of node (tile, c) to LDS, and the pre-squash
// outputs tilde tau_n to tt_node unless it is null.
__device__ __forceinline__ void output_layer(const f32x4 (&acc)[2], LaneTab lt, int w3, int b3, int q,
                                             float* __restrict__ sw_node,
                                             float* __restrict__ tt_node = nullptr) {
    float pn[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        float v = 0.0f;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) v = fmaf(lt[w3 + (u * 4 + r) * 4 + n], acc[u][r], v);
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
        pn[n] = v;
    }
    if (q == 0) {
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            const float t = pn[n] + lt[b3 + n];
            sw_node[n] = 1.0f / (0.5f + 0.5f / (1.0f + expf(t)));
            if (tt_node) tt_node[n] = t;
        }
    }
}

}  // namespace nco
