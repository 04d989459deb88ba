// Energy spectrum E(k) of the velocity field, in float64.
//
// The loss of Sec. "Learning Task" compares shell-summed kinetic energy
// spectra.  Here u_hat = DFT(u) / n^3 over a cubic periodic lattice and
// E(k) = 1/2 sum |u_hat|^2 over the integer wavevectors in [-n/2, n/2)^3 with
// round(|k|) = k.  Lattice sizes such as 96 and 192 are not powers of two: one
// axis at a time, sizes are transformed through up to two factors in LDS
// (below; ft_serves), the largest ones and larger primes by one O(n) dot
// product per output element, register-blocked over 256 frequencies and 8
// lines per wavefront, with a float64 twiddle table.  The velocity is real, so the spectrum readout
// transforms only the half k_x <= n / 2 and counts the conjugate partners
// twice.  The shell sums are deterministic: along a line the shell index never
// decreases with the wavenumber's magnitude, so each (shell, line) sum is one
// run added in order by one thread, and the rest is added in a fixed order.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "kernels.h"

namespace nco {

namespace {

template <int S>
__global__ __launch_bounds__(256) void k_velocity(const typename Codec<S>::store_t* __restrict__ f,
                                                  double* __restrict__ u, int n) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n) return;
    double r = 0, jx = 0, jy = 0, jz = 0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const double v = Codec<S>::to_double(f[(size_t)i * n + idx], i);
        r += v;
        jx += cx_of(i) * v;
        jy += cy_of(i) * v;
        jz += cz_of(i) * v;
    }
    u[idx] = jx / r;
    u[(size_t)n + idx] = jy / r;
    u[2 * (size_t)n + idx] = jz / r;
}

// One axis of the DFT over a [3][n][n][n] field, out[k] = sum_j w^(j k) in[j]
// along AXIS (0 = x, stride 1; 1 = y, stride n; 2 = z, stride n^2) for every
// line ("column") of the field, w = exp(-2 pi i / n), or its conjugate with
// CONJ (the unnormalised inverse).  REAL_IN reads a real field (float64) and
// skips the products with its zero imaginary part.  The x pass computes the
// frequencies k < kout; the y and z passes take only the lines with x < xk
// (kout = xk = n // 2 + 1 for the half spectrum of a real field, n
// otherwise).
//
// Register-blocked: a block of 4 wavefronts takes 32 columns and 256
// frequencies; lane l of wavefront v accumulates the frequencies
// k0 + l + 64 q (q < 4) for the columns 8 v .. 8 v + 7.  The inputs come
// through LDS in chunks of 32 along the axis (loaded once per block, read by
// every lane of a wavefront at the same address, each read feeding four
// frequencies), and a lane's twiddle w^(j k) starts each chunk from the
// table and is advanced by w^k from one j to the next.
constexpr int DB_JC = 32, DB_THREADS = 256;
constexpr int KL = 4, DB_CPW = 8, DB_COLS = 4 * DB_CPW;    // frequencies per lane, columns per wavefront and block

template <int AXIS>
__device__ __forceinline__ size_t dft_stride(int n) {
    return AXIS == 0 ? 1 : AXIS == 1 ? (size_t)n : (size_t)n * n;
}

// Offset of the first element of compact column c (see above): for the x
// pass every x line (c = (comp n + z) n + y); for the y and z passes the
// lines with x < xk, c = (comp n + outer) xk + x, outer = z (y pass) or y
// (z pass).  Column counts stay below 2^32.
template <int AXIS>
__device__ __forceinline__ size_t dft_base(unsigned c, int n, int xk) {
    if constexpr (AXIS == 0) return (size_t)c * n;
    const unsigned q = c / (unsigned)xk, x = c - q * (unsigned)xk;    // q = comp n + outer
    if constexpr (AXIS == 1) return (size_t)q * n * n + x;            // [comp][z][.][x]
    const unsigned comp = q / (unsigned)n, y = q - comp * (unsigned)n;
    return (size_t)comp * n * n * n + (size_t)y * n + x;              // [comp][.][y][x]
}

template <bool REAL_IN>
using dft_elem = typename std::conditional<REAL_IN, double, double2>::type;

// The j loop of one chunk.
template <int AXIS, bool REAL_IN>
__device__ __forceinline__ void dft_chunk(const dft_elem<REAL_IN>* __restrict__ tile, int jn, int wave,
                                          double2 (&w)[KL], const double2 (&wk)[KL],
                                          double2 (&acc)[KL][DB_CPW]) {
#pragma unroll 1
    for (int j = 0; j < jn; ++j) {
#pragma unroll
        for (int c = 0; c < DB_CPW; ++c) {
            const int col = wave * DB_CPW + c;
            const dft_elem<REAL_IN> v = tile[AXIS == 0 ? col * DB_JC + j : j * DB_COLS + col];
#pragma unroll
            for (int q = 0; q < KL; ++q) {
                if constexpr (REAL_IN) {
                    acc[q][c].x = fma(w[q].x, v, acc[q][c].x);
                    acc[q][c].y = fma(w[q].y, v, acc[q][c].y);
                } else {
                    acc[q][c].x = fma(w[q].x, v.x, fma(-w[q].y, v.y, acc[q][c].x));
                    acc[q][c].y = fma(w[q].x, v.y, fma(w[q].y, v.x, acc[q][c].y));
                }
            }
        }
#pragma unroll
        for (int q = 0; q < KL; ++q) {
            const double t = w[q].x * wk[q].x - w[q].y * wk[q].y;
            w[q].y = w[q].x * wk[q].y + w[q].y * wk[q].x;
            w[q].x = t;
        }
    }
}

// Two wavefronts per SIMD (the 128 accumulator registers and a column's
// values in flight).
template <int AXIS, bool REAL_IN, bool CONJ>
__global__ __launch_bounds__(DB_THREADS, 2) void k_dft_axis(
    const void* __restrict__ in_, double2* __restrict__ out, const double2* __restrict__ tw, int n, int kout,
    int xk) {
    // x: [column][j], so that the loads along a line write consecutive LDS
    // words; y, z: [j][column].  Either way a wavefront reads one word.
    __shared__ dft_elem<REAL_IN> tile[DB_JC * DB_COLS];
    const dft_elem<REAL_IN>* __restrict__ in = static_cast<const dft_elem<REAL_IN>*>(in_);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int k0 = blockIdx.y * 64 * KL;
    const unsigned ncol = AXIS == 0 ? 3u * n * n : 3u * n * xk;
    const unsigned c0 = blockIdx.x * DB_COLS;
    const size_t S = dft_stride<AXIS>(n);
    // The loads: x pass, thread t takes j = t % 32 of the columns t / 32 + 8 i;
    // y, z passes, column t % 32 at j = t / 32 + 8 i.
    constexpr int LOADS = DB_JC * DB_COLS / DB_THREADS;
    const int lj = AXIS == 0 ? (int)threadIdx.x % DB_JC : (int)threadIdx.x / DB_COLS;
    const int lc = AXIS == 0 ? (int)threadIdx.x / DB_JC : (int)threadIdx.x % DB_COLS;
    const bool lcol_ok = c0 + lc < ncol;
    const size_t lbase = lcol_ok ? dft_base<AXIS>(c0 + lc, n, xk) : 0;
    double2 acc[KL][DB_CPW];
    double2 w[KL], wk[KL];
    int kq[KL];
#pragma unroll
    for (int q = 0; q < KL; ++q) {
        kq[q] = k0 + lane + 64 * q;
        wk[q] = kq[q] < kout ? tw[kq[q]] : make_double2(1.0, 0.0);
        if constexpr (CONJ) wk[q].y = -wk[q].y;
#pragma unroll
        for (int c = 0; c < DB_CPW; ++c) acc[q][c] = make_double2(0.0, 0.0);
    }
    for (int j0 = 0; j0 < n; j0 += DB_JC) {
        const int jn = min(DB_JC, n - j0);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            dft_elem<REAL_IN> v{};
            if constexpr (AXIS == 0) {
                const int c = lc + (DB_THREADS / DB_JC) * i;
                if (lj < jn && c0 + c < ncol) v = in[(size_t)(c0 + c) * n + j0 + lj];
                tile[c * DB_JC + lj] = v;
            } else {
                const int j = lj + (DB_THREADS / DB_COLS) * i;
                if (j < jn && lcol_ok) v = in[lbase + (size_t)(j0 + j) * S];
                tile[j * DB_COLS + lc] = v;
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < KL; ++q) {
            w[q] = tw[(int)(((long)j0 * (kq[q] < kout ? kq[q] : 0)) % n)];
            if constexpr (CONJ) w[q].y = -w[q].y;
        }
        dft_chunk<AXIS, REAL_IN>(tile, jn, wave, w, wk, acc);
    }
    // Output: the wavefront's 8 columns are consecutive compact columns;
    // their offsets are block-uniform and advance by one line at a time.
    const unsigned cw = c0 + wave * DB_CPW;
    size_t base = cw < ncol ? dft_base<AXIS>(cw, n, xk) : 0;
    unsigned xr = AXIS == 0 ? 0 : cw % (unsigned)xk;       // x of the current line (y, z passes)
    unsigned yr = AXIS == 2 ? (cw / (unsigned)xk) % (unsigned)n : 0;
#pragma unroll
    for (int c = 0; c < DB_CPW; ++c) {
        if (cw + c < ncol)
#pragma unroll
            for (int q = 0; q < KL; ++q)
                if (kq[q] < kout) out[base + (size_t)kq[q] * S] = acc[q][c];
        // Next compact column.
        if constexpr (AXIS == 0) {
            base += n;
        } else {
            if (++xr < (unsigned)xk) {
                base += 1;
            } else if constexpr (AXIS == 1) {
                xr = 0;
                base += (size_t)n * n - (xk - 1);                 // next z (or component)
            } else {
                xr = 0;
                if (++yr < (unsigned)n) {
                    base += (size_t)n - (xk - 1);                 // next y
                } else {
                    yr = 0;
                    base += (size_t)n * n * n - (size_t)(n - 1) * n - (xk - 1);   // next component
                }
            }
        }
    }
}

// Launch of one axis pass over the [3][n][n][n] field (kout, xk as above).
template <int AXIS, bool REAL_IN, bool CONJ = false>
void dft_pass(const void* in, double2* out, const double2* tw, int n, int kout, int xk, hipStream_t st) {
    const size_t ncol = AXIS == 0 ? 3 * (size_t)n * n : 3 * (size_t)n * xk;
    const int kspan = AXIS == 0 ? kout : n;
    const dim3 grid((unsigned)((ncol + DB_COLS - 1) / DB_COLS), (unsigned)((kspan + 64 * KL - 1) / (64 * KL)));
    hipLaunchKernelGGL((k_dft_axis<AXIS, REAL_IN, CONJ>), grid, dim3(DB_THREADS), 0, st, in, out, tw, n, kspan, xk);
}

// The three forward passes: full (every frequency) or the half spectrum
// k_x <= n / 2 of the real velocity field.
void dft_forward(const double* u, double2* A, double2* B, const double2* tw, int n, bool half, hipStream_t st) {
    const int xk = half ? n / 2 + 1 : n;
    dft_pass<0, true>(u, A, tw, n, xk, xk, st);
    dft_pass<1, false>(A, B, tw, n, n, xk, st);
    dft_pass<2, false>(B, A, tw, n, n, xk, st);
}

__device__ __forceinline__ int wavenumber(int idx, int n) { return idx < n - n / 2 ? idx : idx - n; }

// Partial shell sums of one (kz, ky) row; partial is [nbins][n*n], zeroed.
// uh holds k_x = 0 .. n / 2 only (the half spectrum of a real field):
// |u_hat(-k_x, k_y, k_z)| = |u_hat(k_x, -k_y, -k_z)| lies in the same shell,
// so each k_x whose conjugate partner is another k_x counts twice (k_x = 0,
// and -n/2 for even n, once).  The k_x are visited in order of |k_x|, so the
// shell index never decreases along a row.
__global__ __launch_bounds__(256) void k_shell_rows(const double2* __restrict__ uh, int n,
                                                    double* __restrict__ partial, int nbins) {
    const int row = blockIdx.x * blockDim.x + threadIdx.x;
    const int nn = n * n;
    if (row >= nn) return;
    const int kz = wavenumber(row / n, n), ky = wavenumber(row % n, n);
    const size_t n3 = (size_t)n * nn;
    const double scale = 0.5 / ((double)n3 * (double)n3);
    const int c2 = kz * kz + ky * ky;
    int cur = -1;
    double acc = 0.0;
    for (int a = 0; a <= n / 2; ++a) {
        const int b = (int)floor(sqrt((double)(c2 + a * a)) + 0.5);
        if (b != cur) {
            if (cur >= 0 && cur < nbins) partial[(size_t)cur * nn + row] = acc;
            cur = b;
            acc = 0.0;
        }
        const size_t e = (size_t)row * n + a;
        double t = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double2 v = uh[(size_t)c * n3 + e];
            t += (v.x * v.x + v.y * v.y) * scale;
        }
        acc += (a == 0 || 2 * a == n) ? t : 2.0 * t;
    }
    if (cur >= 0 && cur < nbins) partial[(size_t)cur * nn + row] = acc;
}

__global__ __launch_bounds__(256) void k_fill_zero(double* __restrict__ p, size_t count) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0.0;
}

// One block per shell: fixed-order strided sums, a wavefront shuffle
// reduction, then the four wavefront sums in order.
__global__ __launch_bounds__(256) void k_shell_final(const double* __restrict__ partial, int rows,
                                                     double* __restrict__ E) {
    const int b = blockIdx.x;
    double s = 0.0;
    for (int r = threadIdx.x; r < rows; r += blockDim.x) s += partial[(size_t)b * rows + r];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    __shared__ double part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) E[b] = (part[0] + part[1]) + (part[2] + part[3]);
}

// dL/dE at every wavevector: A[c][e] *= dL/dE(shell of e).
__global__ __launch_bounds__(256) void k_scale_shells(double2* __restrict__ A, int n,
                                                      const double* __restrict__ dE, int nbins) {
    const size_t n3 = (size_t)n * n * n;
    const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n3) return;
    const int kx = wavenumber((int)(e % n), n), ky = wavenumber((int)((e / n) % n), n),
              kz = wavenumber((int)(e / ((size_t)n * n)), n);
    const int b = (int)floor(sqrt((double)(kx * kx + ky * ky + kz * kz)) + 0.5);
    const double s = b < nbins ? dE[b] : 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        double2 v = A[(size_t)c * n3 + e];
        v.x *= s;
        v.y *= s;
        A[(size_t)c * n3 + e] = v;
    }
}

// rho and u = j / rho of every node (float64).
template <int S>
__global__ __launch_bounds__(256) void k_rho_u(const typename Codec<S>::store_t* __restrict__ f, double* __restrict__ u,
                                               double* __restrict__ rho, int n) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n) return;
    double r = 0, jx = 0, jy = 0, jz = 0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const double v = Codec<S>::to_double(f[(size_t)i * n + idx], i);
        r += v;
        jx += cx_of(i) * v;
        jy += cy_of(i) * v;
        jz += cz_of(i) * v;
    }
    u[idx] = jx / r;
    u[(size_t)n + idx] = jy / r;
    u[2 * (size_t)n + idx] = jz / r;
    rho[idx] = r;
}

// lambda_f = lambda_rho + c . lambda_j with lambda_u = Re(B) / n^6 (B the
// unnormalised inverse DFT of the shell-weighted spectrum), lambda_j =
// lambda_u / rho, lambda_rho = -lambda_u . u / rho.
__global__ __launch_bounds__(256) void k_lambda_from_u(const double2* __restrict__ B, const double* __restrict__ u,
                                                       const double* __restrict__ rho, int n3, double scale,
                                                       float* __restrict__ lam) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n3) return;
    double lu[3], lr = 0.0;
    const double ir = 1.0 / rho[idx];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        lu[c] = B[(size_t)c * n3 + idx].x * scale;
        lr -= lu[c] * u[(size_t)c * n3 + idx];
    }
    lr *= ir;
#pragma unroll
    for (int i = 0; i < Q; ++i)
        lam[(size_t)i * n3 + idx] = (float)(lr + (cx_of(i) * lu[0] + cy_of(i) * lu[1] + cz_of(i) * lu[2]) * ir);
}

// ---------------------------------------------------- two-factor transform --
//
// One axis of the DFT for n = N1 N2, staged in LDS: with j = N2 j1 + j2 and
// k = k1 + N1 k2,
//   X[k] = sum_j2 w_N2^(j2 k2) ( w_n^(j2 k1) sum_j1 w_N1^(j1 k1) x[j] ),
// N1 + N2 products per output and axis instead of n (32 instead of 256 at
// n = 256).  A thread forms the outputs k1 and N1 - k1 (k2 and N2 - k2) together:
// their factors are conjugate, so the four real products of an input serve
// both.  A block holds C lines of the axis ([j][line], rows of C + 1) and the
// twiddles in LDS.
//
// Passes of the spectrum: the x pass forms the velocity of its rows from the
// populations itself (three lines per row) and writes the half spectrum
// k_x <= n / 2 in rows of n / 2 + 1; the z pass bins |u_hat|^2 into shells in
// LDS and writes one sum per block and shell.  The state is read once
// (1.8 GB at 256^3 in float32) and the half spectrum moves four times (0.4 GB
// each), but what bounds them is their vector instructions: 85-91 % of the issue
// cycles in every pass.  256^3, float32 state: x 0.58-0.67 ms, y 0.28-0.32, z with
// the shells 0.42-0.49, a readout 1.29-1.52 ms where the velocity, direct
// transforms and shells took 4.29 (128^3 0.22 against 0.47, 64^3 0.059 against
// 0.186).
constexpr int FT_THREADS = 512;
constexpr int FT_CAP = 2304;                    // LDS elements of the lines: n (C + 1), 256 x 9
constexpr int FT_SMALL = 256, FT_LARGE = 576;   // twiddles held (two blocks per CU up to 256; 576 (3 + 1) fills FT_CAP)

constexpr int FT_FIELD = -2, FT_REAL = -1;      // line sources; >= 0: populations of that storage

struct FtArgs {
    int n, n1, n2;
    int xk, xs;             // lines x < xk of the y and z passes, row stride of the field
    int kout, ostride;      // x pass: outputs k < kout, row stride of the output
    int lines, c;           // line count (x pass from populations: rows), lines (rows) per block
    int nbins;
};

// Offset of the first element and the stride of line l.
template <int AXIS>
__device__ __forceinline__ size_t ft_base(unsigned l, const FtArgs& a) {
    if constexpr (AXIS == 0) return (size_t)l * a.xs;
    const unsigned q = l / (unsigned)a.xk, x = l - q * (unsigned)a.xk;          // q = comp n + outer
    if constexpr (AXIS == 1) return (size_t)q * a.n * a.xs + x;                 // [comp][z][.][x]
    const unsigned comp = q / (unsigned)a.n, y = q - comp * (unsigned)a.n;
    return (size_t)comp * a.n * a.n * a.xs + (size_t)y * a.xs + x;              // [comp][.][y][x]
}

template <int SRC>
using ft_elem = typename std::conditional<SRC == FT_FIELD, double2, double>::type;

// The outputs p and N - p of an N-point transform over x[m step], m < N, with
// twiddle stride dt per p: (re, im) of both.
template <typename E, bool CONJ>
__device__ __forceinline__ void ft_pair(const E* __restrict__ x, int step, int N, const double2* __restrict__ tw, int dt,
                                        int n, double2& lo, double2& hi) {
    double A = 0.0, B = 0.0, C = 0.0, D = 0.0;
    int w = 0;
#pragma unroll 4
    for (int m = 0; m < N; ++m) {
        const double2 t = tw[w];
        if constexpr (sizeof(E) == sizeof(double2)) {
            const double2 v = x[m * step];
            A = fma(t.x, v.x, A);
            B = fma(t.y, v.y, B);
            C = fma(t.x, v.y, C);
            D = fma(t.y, v.x, D);
        } else {
            const double v = x[m * step];
            A = fma(t.x, v, A);
            D = fma(t.y, v, D);
        }
        w += dt;
        if (w >= n) w -= n;
    }
    if constexpr (CONJ) {
        B = -B;
        D = -D;
    }
    lo = make_double2(A - B, C + D);
    hi = make_double2(A + B, C - D);
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

template <int S> struct CodecOf { using store_t = typename Codec<S>::store_t; };
template <> struct CodecOf<FT_FIELD> { using store_t = double2; };
template <> struct CodecOf<FT_REAL> { using store_t = double; };

template <int AXIS, int SRC, bool CONJ, bool BINS, int TWN>
__global__ __launch_bounds__(FT_THREADS) void k_ft(const void* __restrict__ in_, double2* __restrict__ out,
                                                   const double2* __restrict__ tw_, FtArgs a,
                                                   double* __restrict__ partial) {
    using E = ft_elem<SRC>;
    __shared__ double2 tw[TWN];
    __shared__ E x[FT_CAP];
    __shared__ double2 y[FT_CAP];
    const int tid = threadIdx.x, n = a.n, n1 = a.n1, n2 = a.n2;
    constexpr bool POP = SRC >= 0;
    const int rows0 = blockIdx.x * a.c;                         // first line (row)
    const int nl = (POP ? 3 : 1) * min(a.c, a.lines - rows0);   // lines of this block
    const int cs = (POP ? 3 : 1) * a.c + 1;
    const size_t S = AXIS == 0 ? 1 : AXIS == 1 ? (size_t)a.xs : (size_t)n * a.xs;
    for (int e = tid; e < n; e += FT_THREADS) tw[e] = tw_[e];
    if constexpr (POP) {
        // Velocity of the block's rows, line 3 r + component.
        const auto* __restrict__ f = static_cast<const typename CodecOf<SRC>::store_t*>(in_);
        const int n3 = n * n * n, rows = nl / 3;
        for (int e = tid; e < rows * n; e += FT_THREADS) {
            const int r = e / n, j = e - r * n, idx = (rows0 + r) * n + j;
            double rho = 0, jx = 0, jy = 0, jz = 0;
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                const double v = Codec<SRC>::to_double(f[(size_t)i * n3 + idx], i);
                rho += v;
                jx += cx_of(i) * v;
                jy += cy_of(i) * v;
                jz += cz_of(i) * v;
            }
            x[j * cs + 3 * r] = jx / rho;
            x[j * cs + 3 * r + 1] = jy / rho;
            x[j * cs + 3 * r + 2] = jz / rho;
        }
    } else {
        const E* __restrict__ in = static_cast<const E*>(in_);
        for (int e = tid; e < nl * n; e += FT_THREADS) {
            const int c = AXIS == 0 ? e / n : e % nl, j = AXIS == 0 ? e - c * n : e / nl;
            x[j * cs + c] = in[ft_base<AXIS>(rows0 + c, a) + (size_t)j * S];
        }
    }
    __syncthreads();
    // N1-point transforms over j1 and the twiddle between the factors.
    const int p1 = n1 / 2 + 1, p2 = n2 / 2 + 1;
    for (int t = tid; t < p1 * n2 * nl; t += FT_THREADS) {
        const int q = t / nl, c = t - q * nl, p = q / n2, j2 = q - p * n2;
        double2 lo, hi;
        ft_pair<E, CONJ>(x + j2 * cs + c, n2 * cs, n1, tw, n2 * p, n, lo, hi);
        double2 w = tw[j2 * p];
        if constexpr (CONJ) w.y = -w.y;
        y[(j2 * n1 + p) * cs + c] = cmul(lo, w);
        if (p != 0 && 2 * p != n1) {
            w = tw[j2 * (n1 - p)];
            if constexpr (CONJ) w.y = -w.y;
            y[(j2 * n1 + n1 - p) * cs + c] = cmul(hi, w);
        }
    }
    __syncthreads();
    // N2-point transforms over j2.
    double* __restrict__ en = reinterpret_cast<double*>(x);
    for (int t = tid; t < p2 * n1 * nl; t += FT_THREADS) {
        int c, p, k1;
        if constexpr (AXIS == 0) {
            const int q = t / n1;
            k1 = t - q * n1;
            c = q / p2;
            p = q - c * p2;
            if (k1 + n1 * p >= a.kout && (p == 0 || k1 + n1 * (n2 - p) >= a.kout)) continue;
        } else {
            const int q = t / nl;
            c = t - q * nl;
            p = q / n1;
            k1 = q - p * n1;
        }
        double2 lo, hi;
        ft_pair<double2, CONJ>(y + k1 * cs + c, n1 * cs, n2, tw, n1 * p, n, lo, hi);
        const int k = k1 + n1 * p, kh = k1 + n1 * (n2 - p);
        const bool two = p != 0 && 2 * p != n2;
        if constexpr (BINS) {
            en[k * cs + c] = lo.x * lo.x + lo.y * lo.y;
            if (two) en[kh * cs + c] = hi.x * hi.x + hi.y * hi.y;
        } else if constexpr (AXIS == 0) {
            // Line 3 r + component of row r: [component][row].
            const int l = rows0 + (POP ? c / 3 : c);
            double2* __restrict__ o =
                out + (POP ? (size_t)(c % 3) * a.lines + l : (size_t)l) * a.ostride;
            if (k < a.kout) o[k] = lo;
            if (two && kh < a.kout) o[kh] = hi;
        } else {
            double2* __restrict__ o = out + ft_base<AXIS>(rows0 + c, a);
            o[(size_t)k * S] = lo;
            if (two) o[(size_t)kh * S] = hi;
        }
    }
    if constexpr (BINS) {
        // Shell sums: per line (k_x, k_y) the shells grow with |k_z|, so each
        // (line, shell) is one run of |k_z|, added in order by the thread at
        // its start; then the lines in order.
        static_assert(AXIS == 2 && SRC == FT_FIELD, "the last pass bins");
        double* __restrict__ hist = reinterpret_cast<double*>(y);       // [line][nbins]
        __syncthreads();
        for (int e = tid; e < nl * a.nbins; e += FT_THREADS) hist[e] = 0.0;
        __syncthreads();
        const double scale = 0.5 / ((double)n * n * n * ((double)n * n * n));
        for (int e = tid; e < nl * (n / 2 + 1); e += FT_THREADS) {
            const int kz = e / nl, c = e - kz * nl;
            const unsigned l = rows0 + c, q = l / (unsigned)a.xk;
            const int kx = (int)(l - q * (unsigned)a.xk), ky = wavenumber((int)(q % (unsigned)n), n);
            auto shell = [&](int k) { return (int)floor(sqrt((double)(kx * kx + ky * ky + k * k)) + 0.5); };
            const int b = shell(kz);
            if ((kz > 0 && shell(kz - 1) == b) || b >= a.nbins) continue;
            double s = 0.0;
            for (int k = kz; k <= n / 2 && shell(k) == b; ++k) {
                s += en[k * cs + c];
                if (k > 0 && 2 * k != n) s += en[(n - k) * cs + c];
            }
            hist[c * a.nbins + b] = s * (kx == 0 || 2 * kx == n ? scale : 2.0 * scale);
        }
        __syncthreads();
        for (int b = tid; b < a.nbins; b += FT_THREADS) {
            double s = 0.0;
            for (int c = 0; c < nl; ++c) s += hist[c * a.nbins + b];
            partial[(size_t)b * gridDim.x + blockIdx.x] = s;
        }
    }
}

// The factors of n nearest its square root (n1 >= n2), (n, 1) for a prime.
void ft_factors(int n, int& n1, int& n2) {
    n2 = 1;
    for (int d = 2; d * d <= n; ++d)
        if (n % d == 0) n2 = d;
    n1 = n / n2;
}

// Two-factor transforms serve composite n up to what LDS holds, and primes
// as one factor up to 256: the paired outputs and the fused ends still win
// there (a readout at 67: 0.080 against 0.190 ms of the register-blocked direct
// form, 127: 0.37 against 0.48, 251: 3.5 against 4.1), by less with every
// size; larger primes keep the direct form.  n = 2 p: 326 7.5 against 12.5 ms.
bool ft_serves(int n) {
    int n1, n2;
    ft_factors(n, n1, n2);
    return n <= FT_LARGE && (n2 > 1 || n <= 256);
}

// Lines (rows of three lines) per block: what LDS holds, at most 32 lines,
// fewer where that leaves fewer than 256 blocks (but 8 where possible, for
// full cache lines along x).
int ft_lines(int n, int lines, int per) {
    const int most = std::max(1, std::min(32, FT_CAP / n - 1) / per);
    return std::max(1, std::min(most, std::max((8 + per - 1) / per, (lines + 255) / 256)));
}

FtArgs ft_args(int n, int xk, int xs) {
    FtArgs a{};
    a.n = n;
    ft_factors(n, a.n1, a.n2);
    a.xk = xk;
    a.xs = xs;
    return a;
}

unsigned ft_blocks(const FtArgs& a) { return (unsigned)((a.lines + a.c - 1) / a.c); }

template <int AXIS, int SRC, bool CONJ, bool BINS>
void ft_launch(const void* in, double2* out, const double2* tw, const FtArgs& a, double* partial, hipStream_t st) {
    if (a.n <= FT_SMALL)
        hipLaunchKernelGGL((k_ft<AXIS, SRC, CONJ, BINS, FT_SMALL>), dim3(ft_blocks(a)), dim3(FT_THREADS), 0, st, in, out,
                           tw, a, partial);
    else
        hipLaunchKernelGGL((k_ft<AXIS, SRC, CONJ, BINS, FT_LARGE>), dim3(ft_blocks(a)), dim3(FT_THREADS), 0, st, in, out,
                           tw, a, partial);
}

// One pass over the full [3][n][n][n] field.
template <int AXIS, int SRC, bool CONJ>
void ft_pass(const void* in, double2* out, const double2* tw, int n, hipStream_t st) {
    FtArgs a = ft_args(n, n, n);
    a.kout = a.ostride = n;
    a.lines = 3 * n * n;
    a.c = ft_lines(n, a.lines, 1);
    ft_launch<AXIS, SRC, CONJ, false>(in, out, tw, a, nullptr, st);
}

// E(k) of the populations f (storage S): x, y and z pass, shell sums.
template <int S>
hipError_t ft_spectrum(const void* f, int n, double2* A, double2* B, const double2* tw, double* part, double* E_dev,
                       int nbins, hipStream_t st) {
    const int xk = n / 2 + 1;
    FtArgs a = ft_args(n, xk, xk);
    a.kout = a.ostride = xk;
    a.lines = n * n;
    a.c = ft_lines(n, a.lines, 3);
    ft_launch<0, S, false, false>(f, A, tw, a, nullptr, st);
    a.lines = 3 * n * xk;
    a.c = ft_lines(n, a.lines, 1);
    a.nbins = nbins;
    ft_launch<1, FT_FIELD, false, false>(A, B, tw, a, nullptr, st);
    ft_launch<2, FT_FIELD, false, true>(B, nullptr, tw, a, part, st);
    hipLaunchKernelGGL(k_shell_final, dim3(nbins), dim3(256), 0, st, part, (int)ft_blocks(a), E_dev);
    return hipGetLastError();
}

struct SpecLayout {
    size_t u, a, b, part, tw, rho, total;
};

SpecLayout spec_layout(int n, int nbins) {
    const size_t n3 = (size_t)n * n * n;
    SpecLayout L;
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    L.u = 0;
    L.a = up(L.u + 3 * n3 * sizeof(double));
    L.b = up(L.a + 3 * n3 * sizeof(double2));
    L.part = up(L.b + 3 * n3 * sizeof(double2));
    L.tw = up(L.part + (size_t)nbins * n * n * sizeof(double));
    L.rho = up(L.tw + (size_t)n * sizeof(double2));
    L.total = up(L.rho + n3 * sizeof(double));
    return L;
}

// Twiddles exp(-2 pi i m / n), m = 0 .. n-1, in float64 on the device.
__global__ __launch_bounds__(256) void k_twiddles(double2* __restrict__ tw, int n) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n) return;
    double s, c;
    sincospi(2.0 * (double)m / (double)n, &s, &c);
    tw[m] = make_double2(c, -s);
}

hipError_t upload_twiddles(double2* tw, int n, hipStream_t st) {
    hipLaunchKernelGGL(k_twiddles, dim3((n + 255) / 256), dim3(256), 0, st, tw, n);
    return hipGetLastError();
}

// Scratch of the allocation-free spectrum (nco_energy_spectrum_noalloc):
// one array per device, held until the process ends.  Host code never
// passes the array's name to a kernel (on the host it stands for a host-side
// symbol, not a device address); it uses the device address that
// hipGetSymbolAddress gives, taken once per device with that device current.
constexpr size_t SCRATCH_BYTES = (size_t)36 << 20;
__device__ __align__(256) char scratch[SCRATCH_BYTES];

constexpr int SCRATCH_DEVICES = 64;
void* g_scratch_ptr[SCRATCH_DEVICES] = {};
std::mutex g_scratch_mutex;

}  // namespace

int spectrum_bins(int n) { return (int)floor(sqrt(3.0) * (n / 2) + 0.5) + 1; }

// lam (float [27][n^3]) = (dE/df)^T dL/dE for the spectrum of f; dE lives on
// the device (nbins doubles).  Forward DFT, weight each wavevector by the
// derivative of its shell, inverse DFT, then the chain rule through u = j/rho.
hipError_t launch_spectrum_adjoint(int storage, const void* f, int n, void* work, const double* dE,
                                   int nbins, float* lam, hipStream_t st) {
    const SpecLayout L = spec_layout(n, nbins);
    char* w = static_cast<char*>(work);
    double* u = reinterpret_cast<double*>(w + L.u);
    double2* A = reinterpret_cast<double2*>(w + L.a);
    double2* B = reinterpret_cast<double2*>(w + L.b);
    double2* tw = reinterpret_cast<double2*>(w + L.tw);
    double* rho = reinterpret_cast<double*>(w + L.rho);
    const int n3 = n * n * n;
    if (hipError_t e = upload_twiddles(tw, n, st); e != hipSuccess) return e;
    const int nb = (n3 + 255) / 256;
    switch (storage) {
        case ST_F32: hipLaunchKernelGGL(k_rho_u<ST_F32>, dim3(nb), dim3(256), 0, st, static_cast<const float*>(f), u, rho, n3); break;
        case ST_F16: hipLaunchKernelGGL(k_rho_u<ST_F16>, dim3(nb), dim3(256), 0, st, static_cast<const __half*>(f), u, rho, n3); break;
        case ST_BF16: hipLaunchKernelGGL(k_rho_u<ST_BF16>, dim3(nb), dim3(256), 0, st, static_cast<const __hip_bfloat16*>(f), u, rho, n3); break;
        case ST_F64: hipLaunchKernelGGL(k_rho_u<ST_F64>, dim3(nb), dim3(256), 0, st, static_cast<const double*>(f), u, rho, n3); break;
        default: return hipErrorInvalidValue;
    }
    if (ft_serves(n)) {
        ft_pass<0, FT_REAL, false>(u, A, tw, n, st);
        ft_pass<1, FT_FIELD, false>(A, B, tw, n, st);
        ft_pass<2, FT_FIELD, false>(B, A, tw, n, st);
    } else {
        dft_forward(u, A, B, tw, n, false, st);
    }
    hipLaunchKernelGGL(k_scale_shells, dim3(nb), dim3(256), 0, st, A, n, dE, nbins);
    if (ft_serves(n)) {
        ft_pass<0, FT_FIELD, true>(A, B, tw, n, st);
        ft_pass<1, FT_FIELD, true>(B, A, tw, n, st);
        ft_pass<2, FT_FIELD, true>(A, B, tw, n, st);
    } else {
        dft_pass<0, false, true>(A, B, tw, n, n, n, st);
        dft_pass<1, false, true>(B, A, tw, n, n, n, st);
        dft_pass<2, false, true>(A, B, tw, n, n, n, st);
    }
    const double scale = 1.0 / ((double)n3 * (double)n3);
    hipLaunchKernelGGL(k_lambda_from_u, dim3(nb), dim3(256), 0, st, B, u, rho, n3, scale, lam);
    return hipGetLastError();
}

size_t spectrum_workspace_bytes(int n) { return spec_layout(n, spectrum_bins(n)).total; }

// Bytes of the work space the forward spectrum uses (everything before the
// density array, which only the adjoint needs).
size_t spectrum_forward_bytes(int n) { return spec_layout(n, spectrum_bins(n)).rho; }

size_t spectrum_scratch_bytes() { return SCRATCH_BYTES; }

// Device address of the scratch array on `device` (the current device),
// looked up on the first call per device and kept.
hipError_t spectrum_scratch(int device, void** ptr) {
    if (device < 0 || device >= SCRATCH_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[device]) {
        void* p = nullptr;
        if (hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)); e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[device] = p;
    }
    *ptr = g_scratch_ptr[device];
    return hipSuccess;
}

hipError_t launch_energy_spectrum(int storage, const void* f, int n, void* work, double* E_dev,
                                  int nbins, hipStream_t st) {
    const SpecLayout L = spec_layout(n, nbins);
    char* w = static_cast<char*>(work);
    double* u = reinterpret_cast<double*>(w + L.u);
    double2* A = reinterpret_cast<double2*>(w + L.a);
    double2* B = reinterpret_cast<double2*>(w + L.b);
    double* part = reinterpret_cast<double*>(w + L.part);
    double2* tw = reinterpret_cast<double2*>(w + L.tw);
    const int n3 = n * n * n;
    if (hipError_t e = upload_twiddles(tw, n, st); e != hipSuccess) return e;
    if (ft_serves(n)) {
        switch (storage) {
            case ST_F32: return ft_spectrum<ST_F32>(f, n, A, B, tw, part, E_dev, nbins, st);
            case ST_F16: return ft_spectrum<ST_F16>(f, n, A, B, tw, part, E_dev, nbins, st);
            case ST_BF16: return ft_spectrum<ST_BF16>(f, n, A, B, tw, part, E_dev, nbins, st);
            case ST_F64: return ft_spectrum<ST_F64>(f, n, A, B, tw, part, E_dev, nbins, st);
            default: return hipErrorInvalidValue;
        }
    }
    const int nb = (n3 + 255) / 256;
    switch (storage) {
        case ST_F32: hipLaunchKernelGGL(k_velocity<ST_F32>, dim3(nb), dim3(256), 0, st, static_cast<const float*>(f), u, n3); break;
        case ST_F16: hipLaunchKernelGGL(k_velocity<ST_F16>, dim3(nb), dim3(256), 0, st, static_cast<const __half*>(f), u, n3); break;
        case ST_BF16: hipLaunchKernelGGL(k_velocity<ST_BF16>, dim3(nb), dim3(256), 0, st, static_cast<const __hip_bfloat16*>(f), u, n3); break;
        case ST_F64: hipLaunchKernelGGL(k_velocity<ST_F64>, dim3(nb), dim3(256), 0, st, static_cast<const double*>(f), u, n3); break;
        default: return hipErrorInvalidValue;
    }
    dft_forward(u, A, B, tw, n, true, st);
    const size_t pc = (size_t)nbins * n * n;
    hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)((pc + 255) / 256)), dim3(256), 0, st, part, pc);
    hipLaunchKernelGGL(k_shell_rows, dim3((n * n + 255) / 256), dim3(256), 0, st, A, n, part, nbins);
    hipLaunchKernelGGL(k_shell_final, dim3(nbins), dim3(256), 0, st, part, n * n, E_dev);
    return hipGetLastError();
}

}  // namespace nco
