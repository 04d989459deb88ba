// Spectral modes on the node grid, both ways: the forced modes of a field
// summed over all nodes (analysis) and a field summed over the modes on every
// node (synthesis).  Both factor the phase e^{i k.x} by axes, so that a node
// costs a few multiply-adds per distinct wavenumber of one axis instead of a
// phase per mode.
#pragma once

#include <type_traits>

#include "kernels.h"
#include "stream.h"

namespace nco {

// ------------------------------------------------------------- analysis --
//
// v_hat(k) = sum_x v(x) e^{-i k.x} of a vector field v, per block and mode:
// six doubles (Re, Im of x, y, z) at partial[(6 m + q) nblocks + block].
//
// A block takes up to 256 consecutive x and `rows` consecutive y of one z
// plane (or z of one y plane: ModeGrid).  Thread t keeps to one x (and to the
// rows sub, sub + rp, ...: below 256 nodes per row, rp rows run side by side)
// and accumulates its column's sums of v cos(m y'), v sin(m y') (y' =
// 2 pi y / ny, from a table per block) for the wavenumbers m = |k_y| of the
// modes, MODES_M of them to a group and GROUPS groups to a pass over the
// nodes.  The columns' sums of a group then
// meet the x phases of MODES_K of its modes' wavenumbers |k_x| in LDS, all
// products shared by the modes that need them, and each mode combines four of
// the block's totals with its signs and its z phase.  Which wavenumbers make a
// group, and which |k_x| meet it, is laid out once per set of modes
// (ModeLayout): only those that occur, k_y and k_z modulo ny and nz.
//
// What bounds it: reading the state (the velocity of a 256^3 float32 lattice:
// 1.8 GB), once for up to MODES_M GROUPS distinct |k_y|.  A phase per mode and
// node (about 60 float64 operations each) took 2.07 ms at 256^3 with 16 modes
// and 0.149 ms at 64^3 with 40; contracting the columns once per mode 0.90
// and 0.083 ms; this form 0.35 and 0.013 ms.  A 256^3 step forced in four
// modes of |k_y| 3 to 16: 1.25 ms (2.38 with a phase per mode and node, 2.74
// with every |k_x| and |k_y| up to the largest, three |k_y| to a pass).
constexpr int MODES_M = 3;          // wavenumbers |k_y| per group
constexpr int MODES_K = 3;          // wavenumbers |k_x| per contraction
constexpr int MODES_ROWS = 64;      // rows of the phase table,
constexpr int MODES_ROWS_SHORT = 256;   // and where a block has more (filled anew for every 256)
constexpr int MODES_COLS = 257;     // LDS row of 256 columns
// Groups per pass where there are more than MODES_M distinct |k_y|: what the
// sums' registers allow (18 doubles per group and thread).
constexpr int MODES_GROUPS = 3;

// Blocks of the sums: `width` consecutive x and `rows` consecutive places of
// the other axis of their plane, y, or with `swap` z (the planes are then those
// of one y, and k_y and k_z exchange their parts in all of the above).
struct ModeGrid {
    int nx, n1, n2;             // extents of x, of the rows' axis and of the planes
    bool swap;
    int width, rp, rows, xchunks, ychunks, blocks;
};

// Rows per block: about 16 nodes per thread on large lattices, fewer where
// that would leave fewer than ~500 blocks (64^3: two).  A block costs its
// contractions whatever it holds, and the work space a column per block, so
// the rows go along z where a plane of y holds less than half as many.  BGK
// step forced in the 40 modes of |k| <= 2.5, one block or more per z plane
// against this: 8 x 8 x 16384 431 -> 290 us, 1 x 1 x 262144 3198 -> 402 (a phase
// per mode and node 547 and 524).
inline ModeGrid mode_grid(int nx, int ny, int nz) {
    ModeGrid g;
    g.nx = nx;
    g.width = nx < 256 ? nx : 256;
    g.rp = 256 / g.width;
    const long n = (long)nx * ny * nz;
    long s = n / (256L * 512);
    s = s < 1 ? 1 : s > 16 ? 16 : s;
    const long most = g.rp * s, ry = most < ny ? most : ny, rz = most < nz ? most : nz;
    g.swap = rz >= 2 * ry;
    g.rows = (int)(g.swap ? rz : ry);
    g.n1 = g.swap ? nz : ny;
    g.n2 = g.swap ? ny : nz;
    g.xchunks = (nx + g.width - 1) / g.width;
    g.ychunks = (g.n1 + g.rows - 1) / g.rows;
    g.blocks = g.xchunks * g.ychunks * g.n2;
    return g;
}

// A mode's place in its contraction: among the contraction's |k_x| and the
// group's |k_y|, and the signs of k_x and of k_y modulo ny.
constexpr int mode_place(int mode, int ix, int iy, bool xneg, bool yneg) {
    return mode << 6 | yneg << 5 | xneg << 4 | iy << 2 | ix;
}

// value(idx, p, v): the field's three components v at node idx = (x, y, z) p.
template <int GROUPS, int ROWS, typename F>
__device__ __forceinline__ void mode_partials(F&& value, ModeGrid g, ModeList l, double* __restrict__ partial) {
    constexpr int GROWS = 6 * MODES_M;          // [component 3][m][cos, sin] sums of a column
    constexpr int COMBOS = 3 * MODES_K, PARTS = 256 / COMBOS, VALS = 4 * MODES_M;
    constexpr int YTAB = MODES_M * GROUPS;
    __shared__ double G[GROWS][MODES_COLS], X[2 * MODES_K][MODES_COLS], H[COMBOS * VALS];
    __shared__ Phasor ytab[ROWS][YTAB];
    static_assert(COMBOS * PARTS * VALS <= GROWS * MODES_COLS, "the partial totals reuse G");
    double* const red = &G[0][0];
    const int tid = threadIdx.x, nx = g.nx, ny = g.n1, nz = g.n2;       // y, z: the rows' and the planes' axis
    int b = blockIdx.x;
    const int xc = b % g.xchunks;
    b /= g.xchunks;
    const int y0 = (b % g.ychunks) * g.rows, z = b / g.ychunks;
    const int rows = min(g.rows, ny - y0);
    const int sub = tid / g.width, x = xc * g.width + tid % g.width;
    const bool active = sub < g.rp && x < nx;
    const int nt = g.rp * g.width;              // threads with a column
    const Phasor bx = axis_phasor(active ? x : 0, nx), bz = axis_phasor(z, nz);
    // One contraction of a group, whose column sums are acc.
    auto contract = [&](const ModeChunk& ch, const double(&acc)[3][2 * MODES_M]) __attribute__((always_inline)) {
        ModeEntry next = ch.begin + tid < ch.end ? l.entries[ch.begin + tid] : ModeEntry{0, 0};
        __syncthreads();
#pragma unroll
        for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int j = 0; j < 2 * MODES_M; ++j) G[2 * MODES_M * d + j][tid] = acc[d][j];
#pragma unroll
        for (int k = 0; k < MODES_K; ++k) {
            const Phasor e = phasor_pow(bx, ch.kx[k]);
            X[2 * k][tid] = e.c;
            X[2 * k + 1][tid] = e.s;
        }
        __syncthreads();
        // Thread (k, component, part): its run of columns, the sums
        // [m][cos, sin of y'] x [cos, sin of x'].
        const int combo = tid % COMBOS, part = tid / COMBOS, k = combo % MODES_K, d = combo / MODES_K;
        double t[VALS];
#pragma unroll
        for (int j = 0; j < VALS; ++j) t[j] = 0.0;
        if (part < PARTS) {
            const int c1 = (part + 1) * nt / PARTS;
            for (int c = part * nt / PARTS; c < c1; ++c) {
                const double xcs = X[2 * k][c], xsn = X[2 * k + 1][c];
#pragma unroll
                for (int j = 0; j < 2 * MODES_M; ++j) {
                    const double v = G[2 * MODES_M * d + j][c];
                    t[2 * j] = fma(v, xcs, t[2 * j]);
                    t[2 * j + 1] = fma(v, xsn, t[2 * j + 1]);
                }
            }
        }
        __syncthreads();
        if (part < PARTS)
#pragma unroll
            for (int j = 0; j < VALS; ++j) red[(combo * VALS + j) * PARTS + part] = t[j];
        __syncthreads();
        if (tid < COMBOS * VALS) {
            double s = 0.0;
            for (int q = 0; q < PARTS; ++q) s += red[tid * PARTS + q];
            H[tid] = s;
        }
        __syncthreads();
        for (int i = ch.begin + tid; i < ch.end; i += 256) {
            const int e = next.place, m = e >> 6, ix = e & 3, iy = (e >> 2) & 3;
            const bool xneg = e & 16, yneg = e & 32;
            const Phasor ez = phasor_pow(bz, -next.kz);
            if (i + 256 < ch.end) next = l.entries[i + 256];
            for (int c = 0; c < 3; ++c) {
                // sum of v cos y' cos x', v cos y' sin x', v sin y' cos x', v sin y' sin x'
                const double* h = H + ((c * MODES_K + ix) * VALS + 4 * iy);
                const double sxy = xneg != yneg ? -h[3] : h[3];
                const Phasor o = phasor_mul(Phasor{h[0] - sxy, -((xneg ? -h[1] : h[1]) + (yneg ? -h[2] : h[2]))}, ez);
                partial[(size_t)(6 * m + 2 * c) * gridDim.x + blockIdx.x] = o.c;
                partial[(size_t)(6 * m + 2 * c + 1) * gridDim.x + blockIdx.x] = o.s;
            }
        }
    };
    // The next contraction (they follow one another in the order of the groups),
    // read ahead.
    ModeChunk ch = l.chunk[0];
    int at = 0;
    for (int pass = 0; pass < l.groups; pass += GROUPS) {
        double acc[GROUPS][3][2 * MODES_M];
#pragma unroll
        for (int u = 0; u < GROUPS; ++u)
#pragma unroll
            for (int d = 0; d < 3; ++d)
#pragma unroll
                for (int j = 0; j < 2 * MODES_M; ++j) acc[u][d][j] = 0.0;
        for (int r0 = 0; r0 < rows; r0 += ROWS) {
            const int nr = min(ROWS, rows - r0);
            if (r0 > 0) __syncthreads();
            for (int e = tid; e < nr * YTAB; e += 256) {
                const int j = e % YTAB, gr = pass + j / MODES_M;
                const int m = gr < l.groups ? l.group[gr].ky[j % MODES_M] : 0;
                ytab[e / YTAB][j] = axis_phasor((int)(((long)m * (y0 + r0 + e / YTAB)) % ny), ny);
            }
            __syncthreads();
            if (!active) continue;
            for (int r = sub; r < nr; r += g.rp) {
                const int y = y0 + r0 + r;
                const NodeIdx p = g.swap ? NodeIdx{x, z, y} : NodeIdx{x, y, z};
                double v[3];
                value((g.swap ? p.z * nz + p.y : p.z * ny + p.y) * nx + x, p, v);
#pragma unroll
                for (int j = 0; j < YTAB; ++j) {
                    const Phasor e = ytab[r][j];
                    auto& s = acc[j / MODES_M];
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        s[d][2 * (j % MODES_M)] = fma(v[d], e.c, s[d][2 * (j % MODES_M)]);
                        s[d][2 * (j % MODES_M) + 1] = fma(v[d], e.s, s[d][2 * (j % MODES_M) + 1]);
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < GROUPS; ++u)
            if (pass + u < l.groups)
                for (const int g1 = l.group[pass + u].end;;) {
                    contract(ch, acc[u]);
                    if (++at < l.chunks) ch = l.chunk[at];
                    if (at == g1) break;
                }
        __syncthreads();
    }
}

// Launches launch(groups per pass, rows of the table), both as types, for the
// grid and the list.
template <typename L>
void mode_launch(const ModeGrid& g, const ModeList& l, L&& launch) {
    using One = std::integral_constant<int, 1>;
    using All = std::integral_constant<int, MODES_GROUPS>;
    using Few = std::integral_constant<int, MODES_ROWS>;
    using Many = std::integral_constant<int, MODES_ROWS_SHORT>;
    if (l.groups == 1)
        g.rows <= MODES_ROWS ? launch(One{}, Few{}) : launch(One{}, Many{});
    else
        g.rows <= MODES_ROWS ? launch(All{}, Few{}) : launch(All{}, Many{});
}

// ------------------------------------------------------------ synthesis --
//
// F(x, y, z) = scale sum_m Re(c_m e^{i k_m.x}), separable in x: with
// R_m(y, z) = scale c_m e^{i 2 pi (k_y y / ny + k_z z / nz)},
//   F(x, y, z) = sum_kx Re(S_kx(y, z) e^{i 2 pi kx x / nx}),
//   S_kx(y, z) = sum of R_m over the modes m with k_x = kx (in mode order),
// so a node sums 2 kx_max + 1 terms whatever the number of modes.  A block
// serves SYN_ROWS consecutive (y, z) rows: its threads first form S for each
// (row, kx) in LDS (one sincospi of an exact fraction per mode and row), then
// each node takes its x phase e^{i 2 pi x / nx} (from an LDS table the block
// fills, one sincospi per x) and the powers up to kx_max by products.
// float64 throughout.
constexpr int SYN_ROWS = 8;
constexpr int SYN_CHUNK = 32;
constexpr int SYN_XTAB = 1024;                  // x-phase table in LDS up to this extent

struct SynLds {
    double2 S[SYN_ROWS][2 * FORCE_KX_MAX + 1][3];
    double2 R[SYN_ROWS][SYN_CHUNK][3];
    int skx[SYN_CHUNK];
    double2 xph[SYN_XTAB];                      // e^{i 2 pi x / nx}
};

// S of the block's rows (all threads of a 256-thread block; ends with a
// barrier).  coef[6 m ..]: (Re, Im) of the x, y, z components of c_m.
__device__ __forceinline__ void synthesis_rows(SynLds& l, const StepArgs& a, int kx_max, const double* __restrict__ coef,
                                               double scale) {
    const int row0 = blockIdx.x * SYN_ROWS;
    const int nrows = a.ny * a.nz;
    const int nk = 2 * kx_max + 1;
    if (a.nx <= SYN_XTAB)
        for (int x = threadIdx.x; x < a.nx; x += blockDim.x) {
            double sn, cs;
            sincospi(2.0 * (double)x / (double)a.nx, &sn, &cs);
            l.xph[x] = make_double2(cs, sn);
        }
    for (int e = threadIdx.x; e < SYN_ROWS * nk; e += blockDim.x)
#pragma unroll
        for (int d = 0; d < 3; ++d) l.S[e / nk][e % nk][d] = make_double2(0.0, 0.0);
    for (int m0 = 0; m0 < a.n_modes; m0 += SYN_CHUNK) {
        const int mend = min(SYN_CHUNK, a.n_modes - m0);
        // R_m(row) for every (row, mode) of the chunk, one per thread.
        for (int e = threadIdx.x; e < SYN_ROWS * SYN_CHUNK; e += blockDim.x) {
            const int rr = e / SYN_CHUNK, c = e % SYN_CHUNK, m = m0 + c, row = row0 + rr;
            double2 v[3] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
            if (c < mend && row < nrows) {
                const int y = row % a.ny, z = row / a.ny;
                const int* k = a.fk + 3 * m;
                const long py = ((long)k[1] * y) % a.ny, pz = ((long)k[2] * z) % a.nz;
                const double turn = (double)py / a.ny + (double)pz / a.nz;
                double sn, cs;
                sincospi(2.0 * turn, &sn, &cs);
                const double* fh = coef + 6 * m;
#pragma unroll
                for (int d = 0; d < 3; ++d)
                    v[d] = make_double2(scale * (fh[2 * d] * cs - fh[2 * d + 1] * sn),
                                        scale * (fh[2 * d] * sn + fh[2 * d + 1] * cs));
            }
#pragma unroll
            for (int d = 0; d < 3; ++d) l.R[rr][c][d] = v[d];
        }
        if (threadIdx.x < SYN_CHUNK) l.skx[threadIdx.x] = (int)threadIdx.x < mend ? a.fk[3 * (m0 + threadIdx.x)] : 0;
        __syncthreads();
        // S_kx += the chunk's modes with that k_x, in mode order.
        for (int e = threadIdx.x; e < SYN_ROWS * nk; e += blockDim.x) {
            const int rr = e / nk, kx = e % nk - kx_max;
            double2 acc[3] = {l.S[rr][kx + kx_max][0], l.S[rr][kx + kx_max][1], l.S[rr][kx + kx_max][2]};
            for (int c = 0; c < mend; ++c)
                if (l.skx[c] == kx)
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        acc[d].x += l.R[rr][c][d].x;
                        acc[d].y += l.R[rr][c][d].y;
                    }
#pragma unroll
            for (int d = 0; d < 3; ++d) l.S[rr][kx + kx_max][d] = acc[d];
        }
        __syncthreads();
    }
}

// The field at x of the block's row r.
__device__ __forceinline__ void synthesis_node(const SynLds& l, int nx, int kx_max, int r, int x, double (&F)[3]) {
    double sn, cs;
    if (nx <= SYN_XTAB) {
        sn = l.xph[x].y;
        cs = l.xph[x].x;
    } else {
        sincospi(2.0 * (double)x / (double)nx, &sn, &cs);
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) F[d] = l.S[r][kx_max][d].x;
    double pc = 1.0, ps = 0.0;                  // e^{i k theta}, k = 1 .. kx_max
    for (int k = 1; k <= kx_max; ++k) {
        const double t = pc * cs - ps * sn;
        ps = pc * sn + ps * cs;
        pc = t;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double2 sp = l.S[r][kx_max + k][d], sm = l.S[r][kx_max - k][d];
            // Re(sp e^{i k theta}) + Re(sm e^{-i k theta})
            F[d] += (sp.x + sm.x) * pc - (sp.y - sm.y) * ps;
        }
    }
}

inline unsigned synthesis_blocks(const StepArgs& a) { return (unsigned)((a.ny * a.nz + SYN_ROWS - 1) / SYN_ROWS); }

}  // namespace nco
