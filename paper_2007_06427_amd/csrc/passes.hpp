// The passes of one fictitious-time step of the KS loop dynamics, as block-level device
// functions over one tile of a batch of loops (Sec. 4.2 of Azimi, Ashtari & Schneider,
// arXiv:2007.06427).
//
// Notation: M = Nx and N = Ns grid points. The band is |j| <= Kx and |k| <= Ks, with
// Kx = (M-1)/3 and Ks = (N-1)/3. C = Kx + 1 retained non-negative spatial modes and
// NB = 2 Ks + 1 retained temporal modes. q_j = 2 pi j / L and omega_k = 2 pi k.
//
// Pass A (columns): A(j, s_n) = sum_k u_hat_{j,k} e^{2 pi i n k / N}, an inverse
//                   s-transform of each retained column.
// Pass B (rows):    u at (x_m, s_n) from the inverse x-transform of A(., s_n); u^2 on the
//                   grid; B(j, s_n) = (i q_j / 2) times the forward x-transform of u^2, j < C,
//                   which is the transform of u u_x = (1/2) (u^2)_x. Rows longer than
//                   kSquareMaxM take u_x from a second inverse transform and the product u u_x
//                   instead (accuracy, see kSquareMaxM). (Each transform carries two rows.)
// Pass C (columns): w_hat = forward s-transform of B, then the residual of eq. KS_R,
//                     r_hat = -(i omega/T) u_hat - w_hat + q^2 u_hat - q^4 u_hat.
//                   Per-column partial sums of J and dJ/dT. The linear part of the flow,
//                     G_lin = (-i omega/T - q^2 + q^4) r_hat,
//                   stored as G_lin itself, or, when stepping, folded into the update as
//                     U1 = u_hat + dtau sigma G_lin.
//                   C(j, s_n) = inverse s-transform of i q r_hat (r_x by columns).
// Pass D (rows):    u and r_x at each row, p = u r_x, D(j, s_n) = forward x-transform of p.
//                   The block holding row 0 of a loop finishes J and dJ/dT (and T's update).
// Pass E (columns): p_hat = forward s-transform of D, so G_1 = G_lin - p_hat (eq. KS_G),
//                   or u_hat' = U1 - dtau sigma p_hat when stepping. Optionally it also
//                   runs pass A of the next step on the new column, while it is still in
//                   registers.
//
// u u_x is formed as (1/2) (u^2)_x on rows of up to kSquareMaxM points (the square in physical
// space, the paper's pseudo-spectral treatment of products, and the derivative in spectral
// space) and as the product u * u_x on longer rows; u r_x is always a product in physical space.
// Every product is of band-limited fields on the full grid, so it is free of aliasing inside
// the band, and differentiating the square there is exact. Truncation to the band is implicit:
// only retained modes are ever formed.
//
// Device layouts (complex values, interleaved doubles), one loop after another:
//   band state U, G   [l][j][kk]  j < C, kk < NB: kk = k (k >= 0), kk = k + NB (k < 0)
//   intermediates     [l][j][n]   j < C, n < N
// Columns are contiguous, so column passes read and write whole columns. Row passes stage
// a tile of rows through LDS.
#pragma once

#include "fft.hpp"

namespace lo {

constexpr int kBlock = 256;  // threads per block for every pass kernel

enum Mode : int {
    MODE_RESIDUAL = 0,  // pass C writes r_hat (band layout) into G
    MODE_COST = 1,      // pass C partials only
    MODE_GRAD = 2,      // pass C writes G_lin, pass E turns it into G_1
    MODE_STEP = 3,      // pass C writes U1, pass D advances T, pass E writes u_hat'
    MODE_ADJOINT = 4,   // reverse mode from a saved residual: pass D skips the finalize, pass E
                        // forms G_lin from R and writes scale_l w_j G_1 into G
};

struct Shape {
    int M, N;    // grid points in x and s
    int Kx, Ks;  // band limits
    int H;       // M/2 + 1 columns of the rfft layout
    int C;       // Kx + 1 retained columns
    int NB;      // 2 Ks + 1 retained temporal modes
    int logN;    // log2(N)
    int nloops;
    double L;
};

struct Work {
    cd* A;            // [l][j][n]
    cd* BD;           // [l][j][n]   (B, then D)
    cd* Cb;           // [l][j][n]
    cd* U;            // [l][j][kk]  band state
    cd* G;            // [l][j][kk]  G_lin, U1, r_hat or G_1 depending on the mode
    double* partial;  // [l][j][2]   per-column sums: w_j |r|^2 and w_j Re(u_s conj r)
    double* J;        // [l]
    double* dJdT;     // [l]
    double* Told;     // [l]  period at the start of the current step
    int* status;      // sticky device status
    const cd* R;      // [l][j][kk] saved residual r_hat (MODE_ADJOINT)
    const double* gJ;  // [l] cotangent of J (MODE_ADJOINT; null: all ones)
    const double* dJdT_in;  // [l] dJ/dT of the forward (MODE_ADJOINT)
    double* grad_T;   // [l] gJ dJ/dT, written by pass E (MODE_ADJOINT; null: skipped)
    int herm0;        // U is caller-owned: read column 0 through its Hermitian part
};

// Band index of the temporal partner -k of band index kk (k -> -k).
__device__ __forceinline__ int band_partner(int kk, int NB) { return kk == 0 ? 0 : NB - kk; }

// Band value u[kk] of column j; with herm0, column 0 is read through its Hermitian part
// (u_{0,k} + conj u_{0,-k}) / 2, the part a real field keeps.
__device__ __forceinline__ cd band_get(const cd* u, int j, int kk, int NB, int herm0) {
    const cd v = u[kk];
    if (herm0 && j == 0) {
        const cd w = u[band_partner(kk, NB)];
        return cd{0.5 * (v.x + w.x), 0.5 * (v.y - w.y)};
    }
    return v;
}

constexpr double kTwoPi = 6.283185307179586476925286766559005768;

// compact band index of FFT-order row e, or -1 outside the band
__device__ __forceinline__ int band_row(int e, int N, int Ks) {
    if (e <= Ks) return e;
    if (e >= N - Ks) return e - (N - 2 * Ks - 1);
    return -1;
}

// ---------------------------------------------------------------------------- column passes
// TPF = N/PT threads per column transform, F = kBlock / TPF columns per block, each thread's
// columns and positions from FftPos (its spectrum side: column js, band values at t + m TPF; its
// points side: column jt, s-grid points point(m)). Column c = block * F + f runs over
// nloops * C columns, loop-major. Every column length takes 8 points per thread: a
// 1024-point column spans two wavefronts. 16 points per thread, one wavefront per column,
// measured slower on 64 loops of 256 x 1024 (pass C 57.8 against 52.8 us, the reverse pass's
// column pass 79.9 against 73.9 us): the LDS of a column is the same, so a CU holds the same
// columns, on half the wavefronts.
__host__ __device__ constexpr int col_pt(int) { return 8; }
__host__ __device__ constexpr int col_per_block(int N) { return kBlock / (N / col_pt(N)); }

template <int N>
struct ColG {
    static constexpr int PT = col_pt(N);
    static constexpr int TPF = N / PT;
    static constexpr int F = kBlock / TPF;
    static constexpr int LDS = F * Fft<N, PT>::XS;  // complex values of exchange space per block
};

// Per-column sum over the TPF threads of each transform (spectrum side), in a fixed order.
// Within a wavefront this is an xor tree. A transform that spans two wavefronts adds the two
// wavefront sums through `red` (2 kBlock/64 doubles of LDS), lower wavefront first.
template <int N>
__device__ __forceinline__ void col_sum2(double& a, double& b, double* red) {
    using G = ColG<N>;
    if constexpr (Fft<N, G::PT>::L == 1) {  // a transform's threads are the lanes equal modulo 64 / TPF
        a = sum_lanes<32, 64 / G::TPF>(a);
        b = sum_lanes<32, 64 / G::TPF>(b);
    } else {
        constexpr int W = G::TPF < 64 ? G::TPF : 64;
        a = sum_lanes<W / 2>(a);
        b = sum_lanes<W / 2>(b);
    }
    if constexpr (G::TPF > 64) {
        static_assert(G::TPF == 128, "transforms span at most two wavefronts");
        const int wave = threadIdx.x / 64;
        if (threadIdx.x % 64 == 0) {
            red[2 * wave] = a;
            red[2 * wave + 1] = b;
        }
        __syncthreads();
        const int w0 = wave & ~1;
        a = red[2 * w0] + red[2 * w0 + 2];
        b = red[2 * w0 + 1] + red[2 * w0 + 3];
        __syncthreads();
    }
}

// The columns of a thread. Spectrum side: active, loop l, column j, position t. Points side:
// whether its column exists, and the column's first point within the thread's slots.
template <int N>
struct ColPos {
    using G = ColG<N>;
    FftPos<N, G::PT> p;
    bool active, active_t;
    int l, j, t;
    size_t col_t;  // column index of the points side
    __device__ __forceinline__ ColPos(const Shape& sh, int block) : p(threadIdx.x) {
        const int c = block * G::F + p.xs, n = sh.nloops * sh.C;
        t = p.t;
        active = c < n;
        l = active && sh.nloops > 1 ? c / sh.C : 0;
        j = active ? c - l * sh.C : 0;
        const int ct = block * G::F + p.xt;
        active_t = ct < n;
        col_t = active_t ? ct : 0;
    }
};

// Slot m of a column's spectrum, e = t + m TPF: whether it lies in the band, its band index kk
// and signed mode k. N fixes the band limit, so most slots are resolved at compile time: only the
// two that straddle an edge of the band test t. The column passes of the step are bound by
// vector instructions and memory about equally; with the index arithmetic gone, fused
// multiply-adds in the band functions below and one division per mode instead of two (pass E),
// pass C of 64 loops of 256 x 1024 took 64 us instead of 75 and pass E with the next A 58
// instead of 69.
template <int N, int m>
struct BandSlot {
    static constexpr int TPF = ColG<N>::TPF, Ks = (N - 1) / 3, NB = 2 * Ks + 1;
    static constexpr int lo = m * TPF, hi = lo + TPF - 1;
    static constexpr bool neg = lo >= N / 2;
    static constexpr bool out = lo > Ks && hi < N - Ks;
    static constexpr bool full = hi <= Ks || lo >= N - Ks;
    static __device__ __forceinline__ bool in(int t) {
        return !out && (full || (neg ? lo + t >= N - Ks : lo + t <= Ks));
    }
    static __device__ __forceinline__ int kk(int t) { return neg ? lo + t - (N - NB) : lo + t; }
    static __device__ __forceinline__ int k(int t) { return neg ? lo + t - N : lo + t; }
};

// The band values of this thread's slots of column (l, j) (zero outside the band or for an
// inactive column), read through band_get. Column passes issue these loads before their
// transforms, so that their latency overlaps the transform instead of following it.
template <int N>
__device__ __forceinline__ void band_prefetch(const ColPos<N>& p, const cd* u, int herm0, cd* out) {
    static_for<ColG<N>::PT>([&](auto mc) {
        using B = BandSlot<N, decltype(mc)::value>;
        out[mc] = (p.active && B::in(p.t)) ? band_get(u, p.j, B::kk(p.t), B::NB, herm0) : cd{0.0, 0.0};
    });
}

// The spectral factors of column j, q = 2 pi j / L.
struct ColCoef {
    double q;
    double c;     // q^2 - q^4, of -d_xx - d_xxxx
    double lamx;  // -q^8 + 2 q^6 - q^4, the x part of lambda
    __device__ __forceinline__ ColCoef(int j, double L) {
        q = kTwoPi * j / L;
        const double q2 = q * q, q4 = q2 * q2;
        c = q2 - q4;
        lamx = -q4 * q4 + 2.0 * q4 * q2 - q4;
    }
};

// The residual (eq. KS_R) of mode (j, k): r = -(i om/T) u - (u u_x)_hat + (q^2 - q^4) u, with a =
// om / T and w = N (u u_x)_hat. Every form of the step and of the gradient forms its band values
// through these functions, so that they agree bit for bit.
__device__ __forceinline__ cd band_residual(const ColCoef& f, double a, double invN, cd u, cd w) {
    return cd{__builtin_fma(-invN, w.x, __builtin_fma(a, u.y, f.c * u.x)),
              __builtin_fma(-invN, w.y, __builtin_fma(-a, u.x, f.c * u.y))};
}
// G_lin = (-i om/T - q^2 + q^4) r
__device__ __forceinline__ cd band_glin(const ColCoef& f, double a, cd r) {
    return cd{__builtin_fma(a, r.y, -(f.c * r.x)), __builtin_fma(-a, r.x, -(f.c * r.y))};
}
// dtau sigma: sigma = 1 (explicit) or 1 / (1 - dtau lambda), lambda = lamx - (om/T)^2
__device__ __forceinline__ double band_step(const ColCoef& f, double a, double dtau, int scheme) {
    return scheme ? dtau / __builtin_fma(dtau, __builtin_fma(a, a, -f.lamx), 1.0) : dtau;
}
// G_1 = G_lin - p_hat and u_hat' = U1 - dtau sigma p_hat, p = N p_hat, p_hat = (u r_x)_hat; s =
// dtau sigma / N (N is a power of two: the division is exact)
__device__ __forceinline__ cd band_g1(cd gl, cd p, double invN) {
    return cd{__builtin_fma(-invN, p.x, gl.x), __builtin_fma(-invN, p.y, gl.y)};
}
__device__ __forceinline__ cd band_update(cd u1, cd p, double s) {
    return cd{__builtin_fma(-s, p.x, u1.x), __builtin_fma(-s, p.y, u1.y)};
}
// Adds |r|^2 to J and Re(u_s conj r), u_s = i om u, to dT.
__device__ __forceinline__ void band_sums(double om, cd u, cd r, double& J, double& dT) {
    J = __builtin_fma(r.x, r.x, __builtin_fma(r.y, r.y, J));
    dT = __builtin_fma(om, __builtin_fma(u.x, r.y, -(u.y * r.x)), dT);
}

// The s-grid values of this thread's slots of its points-side column of X.
template <int N>
__device__ __forceinline__ void col_load(const ColPos<N>& p, const cd* X, cd* v) {
    using G = ColG<N>;
    const cd* x = X + p.col_t * N;
#pragma unroll
    for (int m = 0; m < G::PT; ++m) v[m] = p.active_t ? x[p.p.point(m)] : cd{0.0, 0.0};
}

// Inverse s-transform of band column values v (already zero outside the band) into X.
template <int N>
__device__ __forceinline__ void col_inverse_store(const ColPos<N>& p, cd* v, cd* X, cd* ex,
                                                  const TwCache<N, ColG<N>::PT>& twc) {
    using G = ColG<N>;
    fft_inv<N, G::PT>(v, ex, twc, p.p);
    if (p.active_t) {
        cd* x = X + p.col_t * N;
#pragma unroll
        for (int m = 0; m < G::PT; ++m) x[p.p.point(m)] = v[m];
    }
}

template <int N>
__device__ __forceinline__ void col_pass_A(const Shape& sh, int block, const Work& w, cd* ex,
                                           const cd* __restrict__ tw) {
    using G = ColG<N>;
    const ColPos<N> p(sh, block);
    TwCache<N, G::PT> twc;
    tw_cache_load<N, G::PT>(twc, p.p, tw);
    const cd* u = w.U + ((size_t)p.l * sh.C + p.j) * sh.NB;
    cd v[G::PT];
    band_prefetch<N>(p, u, w.herm0, v);
    col_inverse_store<N>(p, v, w.A, ex, twc);
}

// Reverse mode, first pass: the inverse s-transforms of u_hat (into A, as pass A) and of
// i q r_hat from the saved residual (into C, as pass C would leave it), column by column.
// Without WITH_U, A holds u on the s grid already (saved by the forward) and only the
// residual is transformed.
template <int N, bool WITH_U = true>
__device__ __forceinline__ void col_pass_AC(const Shape& sh, int block, const Work& w, cd* ex,
                                            const cd* __restrict__ tw) {
    using G = ColG<N>;
    const ColPos<N> p(sh, block);
    TwCache<N, G::PT> twc;
    tw_cache_load<N, G::PT>(twc, p.p, tw);
    const size_t col = (size_t)p.l * sh.C + p.j;
    const cd* r = w.R + col * sh.NB;
    const double q = kTwoPi * p.j / sh.L;
    cd v[G::PT], rv[G::PT];
    band_prefetch<N>(p, r, 0, rv);  // with WITH_U, in flight during the first transform
    if constexpr (WITH_U) {
        band_prefetch<N>(p, w.U + col * sh.NB, w.herm0, v);
        col_inverse_store<N>(p, v, w.A, ex, twc);
    }
#pragma unroll
    for (int m = 0; m < G::PT; ++m) v[m] = cd{-q * rv[m].y, q * rv[m].x};  // i q r (zero outside the band)
    col_inverse_store<N>(p, v, w.Cb, ex, twc);
}

template <int N>
__device__ __forceinline__ void col_pass_C(const Shape& sh, int block, const double* __restrict__ T, const Work& w,
                                           int mode, double dtau, int scheme, cd* ex, double* red,
                                           const cd* __restrict__ tw) {
    using G = ColG<N>;
    const ColPos<N> p(sh, block);
    const size_t col = (size_t)p.l * sh.C + p.j;
    cd v[G::PT], ub[G::PT];
    col_load<N>(p, w.BD, v);
    band_prefetch<N>(p, w.U + col * sh.NB, w.herm0, ub);  // in flight during the transform
    TwCache<N, G::PT> twc;
    tw_cache_load<N, G::PT>(twc, p.p, tw);
    fft_fwd<N, G::PT>(v, ex, twc, p.p);

    const double invT = 1.0 / (p.active ? T[p.l] : 1.0);
    const ColCoef f(p.j, sh.L);
    constexpr double invN = 1.0 / N;
    double Jp = 0.0, dTp = 0.0;
    cd* g = w.G + col * sh.NB;
    static_for<G::PT>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        using B = BandSlot<N, m>;
        cd x{0.0, 0.0};
        if (p.active && B::in(p.t)) {
            const double om = kTwoPi * B::k(p.t), a = om * invT;
            const cd r = band_residual(f, a, invN, ub[m], v[m]);
            band_sums(om, ub[m], r, Jp, dTp);
            if (mode == MODE_RESIDUAL) {
                g[B::kk(p.t)] = r;
            } else if (mode >= MODE_GRAD) {
                cd gl = band_glin(f, a, r);
                if (mode == MODE_STEP) {
                    const double s = band_step(f, a, dtau, scheme);
                    gl = cd{__builtin_fma(s, gl.x, ub[m].x), __builtin_fma(s, gl.y, ub[m].y)};  // U1
                }
                g[B::kk(p.t)] = gl;
            }
            x = cd{-f.q * r.y, f.q * r.x};  // i q r
        }
        v[m] = x;
    });
    const double wj = (p.j == 0) ? 1.0 : 2.0;
    Jp *= wj;
    dTp *= wj;
    col_sum2<N>(Jp, dTp, red);
    if (p.active && p.t == 0) {
        w.partial[2 * col] = Jp;
        w.partial[2 * col + 1] = dTp;
    }
    if (mode >= MODE_GRAD) col_inverse_store<N>(p, v, w.Cb, ex, twc);
}

template <int N>
__device__ __forceinline__ void col_pass_E(const Shape& sh, int block, const Work& w, int mode, double dtau,
                                           int scheme, bool fuseA, cd* ex, const cd* __restrict__ tw,
                                           const double* __restrict__ T = nullptr) {
    using G = ColG<N>;
    const ColPos<N> p(sh, block);
    const size_t col = (size_t)p.l * sh.C + p.j;
    cd v[G::PT], gb[G::PT];
    col_load<N>(p, w.BD, v);
    // G_lin or (reverse mode) the saved residual, in flight during the transform. In the step
    // (U1, then the next step's pass A on the new column) the loads issued after the transform
    // measured faster: pass E at 256 x 1024 took 70.4 us against 75.8 with them in flight.
    if (mode != MODE_STEP) band_prefetch<N>(p, (mode == MODE_ADJOINT ? w.R : w.G) + col * sh.NB, 0, gb);
    TwCache<N, G::PT> twc;
    tw_cache_load<N, G::PT>(twc, p.p, tw);
    fft_fwd<N, G::PT>(v, ex, twc, p.p);
    if (mode == MODE_STEP) band_prefetch<N>(p, w.G + col * sh.NB, 0, gb);

    constexpr double invN = 1.0 / N;
    const ColCoef f(p.j, sh.L);
    const double invT =
        1.0 / ((mode == MODE_STEP && p.active) ? w.Told[p.l] : (mode == MODE_ADJOINT && p.active) ? T[p.l] : 1.0);
    // reverse mode: G_1 scaled by -gJ_l w_j L, the gradient of sum_l gJ_l J_l in torch's
    // complex convention (gJ folded in by the caller as scale_l = -gJ_l L)
    const double sc = (mode == MODE_ADJOINT && p.active) ? (w.gJ ? -w.gJ[p.l] : -1.0) * sh.L * (p.j == 0 ? 1.0 : 2.0)
                                                         : 1.0;
    cd* g = w.G + col * sh.NB;
    cd* u = w.U + col * sh.NB;
    if (mode == MODE_ADJOINT && w.grad_T && p.active && p.j == 0 && p.t == 0)
        w.grad_T[p.l] = (w.gJ ? w.gJ[p.l] : 1.0) * w.dJdT_in[p.l];
    static_for<G::PT>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        using B = BandSlot<N, m>;
        cd x{0.0, 0.0};
        if (p.active && B::in(p.t)) {
            const double a = kTwoPi * B::k(p.t) * invT;
            if (mode == MODE_ADJOINT) {
                // G_lin as pass C forms it, then G_1 = G_lin - p_hat, p_hat = (u r_x)_hat
                const cd g1 = band_g1(band_glin(f, a, gb[m]), v[m], invN);
                g[B::kk(p.t)] = cd{sc * g1.x, sc * g1.y};
            } else if (mode == MODE_STEP) {
                x = band_update(gb[m], v[m], band_step(f, a, dtau, scheme) * invN);
                u[B::kk(p.t)] = x;
            } else {
                g[B::kk(p.t)] = band_g1(gb[m], v[m], invN);
            }
        }
        v[m] = x;
    });
    if (mode == MODE_STEP && fuseA) col_inverse_store<N>(p, v, w.A, ex, twc);
}

// ---------------------------------------------------------------------------- row passes
// TPF = M/PT threads per row transform, P = kBlock / TPF pairs of rows per block, each
// thread's pairs and positions from FftPos. A block covers ROWS = 2P consecutive global rows
// g0 .. g0 + 2P - 1 (g = l * N + n, loop-major), paired as (g0 + p, g0 + P + p).
//
// Every transform carries the two rows of a pair, f + i g, so its spectrum Z = F + i G over the
// signed frequencies |e| <= Kx is all that passes between memory and the transform. On the
// way in, the thread that loads F_j and G_j forms Z_j and Z_{-j} = conj F_j + i conj G_j and
// stages them in LDS in the order the transform reads them; on the way out, the transforms
// leave Z in LDS and the thread that stores row values reads Z_j and Z_{-j} and splits them. The
// LDS write port is what the row passes run out of first (fft.hpp), and this takes 6 + 6 b128
// writes per thread and field besides the exchange, against 6 (raw tile) + 8 (Z) + 6 (output
// tile) when the rows were staged as separate half spectra: on 64 loops of 256 x 1024 pass B went
// from 64.4 to 54.0 us and pass D from 72.7 to 62.0 (with the exchanges of fft.hpp).
template <int M, int PT_ = (M >= 1024 ? 16 : 8)>
struct RowG {
    static constexpr int PT = PT_, ROW_M = M;
    using E = Fft<M, PT>;
    static constexpr int TPF = M / PT;  // <= 64: one transform per wavefront at most
    static constexpr int P = kBlock / TPF;
    static constexpr int ROWS = 2 * P;
    static constexpr int Kx = (M - 1) / 3;
    static constexpr int CMAX = Kx + 1;
    static constexpr int PW = E::XPW;  // pairs per wavefront
    // Staged spectrum of a pair: frequency e at e (e <= Kx) or e - SH (e >= M - Kx). Strides of a
    // pair (ST) and of a wavefront's region (a multiple of 16 plus WMOD) put 16 consecutive
    // lanes of a staging write (consecutive pairs, then j) on 16 different slots modulo 16.
    static constexpr int SH = M - 2 * Kx - 1;
    static constexpr int up_to(int n, int mod, int r) { return n + ((r - n) % mod + mod) % mod; }
    static constexpr int ST = P >= 16 ? 2 * Kx + 1 : P == 8 ? up_to(2 * Kx + 1, 16, 2) : up_to(2 * Kx + 1, 16, 4);
    static constexpr int WMOD = M == 64 ? 8 : 4;
    static constexpr int wave_region(int fields) {
        const int st = fields * PW * ST, xs = E::L == 1 ? 0 : PW * E::XS;
        return up_to(st > xs ? st : xs, 16, WMOD);
    }
    static constexpr int LDS = kBlock / 64 * wave_region(2);    // two fields (pass D)
    static constexpr int LDS_B = kBlock / 64 * wave_region(1);  // one field (pass B)
    static constexpr int NL = (P * CMAX + kBlock - 1) / kBlock;  // (pair, j) items per thread
    // raw tiles [j][r] of the load unit's copies (load_rows_lds)
    static constexpr int TS = ROWS + 1;
    static constexpr int TILE = CMAX * TS;
};

// Rows of 32 to 512 points keep the twiddle powers (TwCache): they are bound by the vector units'
// issue rate, and the registers cost them no wavefront (pass B of 64 loops of 256 x 1024 went
// from 137 to 168, three wavefronts per SIMD either way, and from 54.3 us to 49.5; pass D 59.7
// to 58.7; pass B of 32-point rows holds 92 so, 110 when each transform forms them, five and four
// wavefronts: a step of 256 ragged loops 38.6 and 40.1 us). Eight points per thread; the 1024-point rows hold 16 and have no registers left.
template <int M, int PT = RowG<M>::PT>
constexpr bool kRowAll = PT == 8 && M >= 32 && M <= 512;

// Item k of a thread: pair p and column j, consecutive lanes on consecutive pairs.
template <class G>
__device__ __forceinline__ bool row_item(int k, int& p, int& j) {
    const int i = threadIdx.x + k * kBlock;
    p = i % G::P;
    j = i / G::P;
    return G::P * G::CMAX % kBlock == 0 || j < G::CMAX;
}

// Staging slot of (pair p, field q) in regions of WR values per wavefront.
template <class G, int WR>
__device__ __forceinline__ int stage_base(int p, int q) {
    return p / G::PW * WR + (q * G::PW + p % G::PW) * G::ST;
}

// Address of column 0 of global row g; element j follows at j * sh.N (intermediates in HBM).
__device__ __forceinline__ size_t row_offset(size_t g, const Shape& sh) {
    return ((g >> sh.logN) * sh.C) * sh.N + (g & (size_t)(sh.N - 1));
}

// The rows of NT intermediates X[0..NT) for this thread's items: issue() puts every global load
// in flight (into registers), commit() stages them as packed spectra. Rows past nrows read as
// zero. ROWS and N are powers of two and tiles start at multiples of ROWS, so when N >= ROWS a
// tile lies inside one loop and its elements sit at j N + r from the tile's first row (32-bit
// offsets); shorter loops take the general row-by-row address.
template <class G, int NT>
struct RowLoad {
    cd fa[NT][G::NL], fb[NT][G::NL];
    __device__ __forceinline__ void issue(const cd* const (&X)[NT], size_t g0, const Shape& sh, size_t nrows) {
        const bool in_loop = sh.N >= G::ROWS;
        const size_t base = row_offset(g0, sh);
#pragma unroll
        for (int k = 0; k < G::NL; ++k) {
            int p, j;
            const bool item = row_item<G>(k, p, j);
            const size_t ga = g0 + p, gb = ga + G::P;
            const bool oka = item && ga < nrows, okb = item && gb < nrows;
            const size_t a = in_loop ? base + (j * sh.N + p) : oka ? row_offset(ga, sh) + (size_t)j * sh.N : 0;
            const size_t b = in_loop ? base + (j * sh.N + G::P + p) : okb ? row_offset(gb, sh) + (size_t)j * sh.N : 0;
#pragma unroll
            for (int q = 0; q < NT; ++q) {
                fa[q][k] = oka ? X[q][a] : cd{0.0, 0.0};
                fb[q][k] = okb ? X[q][b] : cd{0.0, 0.0};
            }
        }
    }
    template <int WR>
    __device__ __forceinline__ void commit(cd* lds) const {
#pragma unroll
        for (int k = 0; k < G::NL; ++k) {
            int p, j;
            if (!row_item<G>(k, p, j)) continue;
#pragma unroll
            for (int q = 0; q < NT; ++q) {
                cd* z = lds + stage_base<G, WR>(p, q);
                const cd f = fa[q][k], g = fb[q][k];
                if (j == 0) {
                    z[0] = cd{f.x, g.x};  // X_0 is read as real
                } else {
                    z[j] = cd{f.x - g.y, f.y + g.x};
                    z[G::ROW_M - G::SH - j] = cd{f.x + g.y, g.x - f.y};
                }
            }
        }
    }
};

// The staged spectrum of a pair (field base z) in the slots of thread t; slots outside the
// band are zero. A slot wholly inside or outside the band is resolved at compile time.
template <class G, int m = 0>
__device__ __forceinline__ void row_gather(const cd* z, int t, cd* v) {
    if constexpr (m < G::PT) {
        constexpr int lo = m * G::TPF, hi = lo + G::TPF - 1;
        constexpr int Kx = G::Kx, M = G::ROW_M;
        if constexpr (hi <= Kx) {
            v[m] = z[lo + t];
        } else if constexpr (lo >= M - Kx) {
            v[m] = z[lo + t - G::SH];
        } else if constexpr (lo > Kx && hi < M - Kx) {
            v[m] = cd{0.0, 0.0};
        } else {
            const int e = lo + t;
            const bool pos = e <= Kx, in = pos || e >= M - Kx;
            const cd x = z[in ? (pos ? e : e - G::SH) : 0];
            v[m] = in ? x : cd{0.0, 0.0};
        }
        row_gather<G, m + 1>(z, t, v);
    }
}

// The reverse: the in-band slots of a transform's output into the staged layout.
template <class G, int m = 0>
__device__ __forceinline__ void row_put(cd* z, int t, const cd* v) {
    if constexpr (m < G::PT) {
        constexpr int lo = m * G::TPF, hi = lo + G::TPF - 1;
        constexpr int Kx = G::Kx, M = G::ROW_M;
        if constexpr (hi <= Kx) {
            z[lo + t] = v[m];
        } else if constexpr (lo >= M - Kx) {
            z[lo + t - G::SH] = v[m];
        } else if constexpr (!(lo > Kx && hi < M - Kx)) {
            const int e = lo + t;
            if (e <= Kx) z[e] = v[m];
            if (e >= M - Kx) z[e - G::SH] = v[m];
        }
        row_put<G, m + 1>(z, t, v);
    }
}

// Split of Z = W_a + i W_b at +-j into the half spectra of rows a and b: W_a(j) = (Z_j + conj
// Z_{-j}) / 2, W_b(j) = (Z_j - conj Z_{-j}) / (2i), scaled by 1/M. With DX they are
// differentiated on the way, i q_j / 2 W (the half derivative of a square).
template <int M, bool DX>
__device__ __forceinline__ void row_split(double L, int j, cd a, cd b, cd& wa, cd& wb) {
    if constexpr (DX) {
        const double c = (kTwoPi / L) * (0.25 / M) * j;  // q_j / 2 and the 1/(2M) of the split
        wa = cd{c * (b.y - a.y), c * (a.x + b.x)};
        wb = cd{c * (a.x - b.x), c * (a.y + b.y)};
    } else {
        constexpr double s = 0.5 / M;
        wa = cd{(a.x + b.x) * s, (a.y - b.y) * s};
        wb = cd{(a.y + b.y) * s, (b.x - a.x) * s};
    }
}

// Rows of the products from the staged spectra (regions of WR values per wavefront) to X.
template <class G, int WR, bool DX>
__device__ __forceinline__ void row_store(const cd* lds, cd* X, size_t g0, const Shape& sh, size_t nrows) {
    const bool in_loop = sh.N >= G::ROWS;
    const size_t base = row_offset(g0, sh);
#pragma unroll
    for (int k = 0; k < G::NL; ++k) {
        int p, j;
        if (!row_item<G>(k, p, j)) continue;
        const cd* z = lds + stage_base<G, WR>(p, 0);
        const cd a = z[j], b = z[j == 0 ? 0 : G::ROW_M - G::SH - j];
        cd wa, wb;
        row_split<G::ROW_M, DX>(sh.L, j, a, b, wa, wb);
        const size_t ga = g0 + p, gb = ga + G::P;
        if (ga < nrows) X[in_loop ? base + (j * sh.N + p) : row_offset(ga, sh) + (size_t)j * sh.N] = wa;
        if (gb < nrows) X[in_loop ? base + (j * sh.N + G::P + p) : row_offset(gb, sh) + (size_t)j * sh.N] = wb;
    }
}

// The rows that RowLoad stages, as raw tiles copied by the load unit straight into LDS
// (global_load_lds_dwordx4: lane i of a wavefront writes 16 bytes at the instruction's LDS
// base + 16 i). One wavefront instruction moves 64 consecutive rows of one column j to
// tile[j][r0 .. r0 + 63], so ROWS must be a multiple of 64. Nothing passes through vector
// registers. Lanes whose row lies past nrows store zeros with ordinary LDS writes instead.
// With WAIT the wavefront waits for its own copies before returning (otherwise the caller
// waits for vmcnt(0) itself); the caller's barrier then makes every wavefront's copies
// visible to the block.
template <int ROWS, int CMAX, int TS, int TILE, int NT, bool WAIT = true>
__device__ __forceinline__ void load_rows_lds(cd* tile, const cd* const (&X)[NT], size_t g0, const Shape& sh,
                                              size_t nrows) {
    static_assert(ROWS % 64 == 0, "a copy instruction covers 64 rows of one column");
    constexpr int RC = ROWS / 64;
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    constexpr int per_field = CMAX * RC;
    const size_t g = g0 + lane;
    for (int k = wave; k < NT * per_field; k += kBlock / 64) {
        const int q = k / per_field, rem = k % per_field;
        const int j = rem / RC, r0 = (rem % RC) * 64;
        cd* dst = tile + q * TILE + j * TS + r0;
        const size_t gr = g + r0;
        if (gr < nrows) {
            const cd* src = X[q] + ((gr >> sh.logN) * CMAX + j) * sh.N + (gr & (size_t)(sh.N - 1));
            __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void*)const_cast<cd*>(src),
                                             (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
        } else {
            dst[lane] = cd{0.0, 0.0};
        }
    }
    if constexpr (WAIT) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// F + i G of rows ra (F) and rb (G) of an array X[j][r] (stride ld) of half spectra, in the slots of thread
// t; slots outside the band are zero. B_ROW false: row b is empty. The values are those that
// RowLoad stages.
template <class G, bool B_ROW, int m = 0>
__device__ __forceinline__ void row_gather_raw(const cd* X, int ld, int ra, int rb, int t, cd* v) {
    if constexpr (m < G::PT) {
        constexpr int lo = m * G::TPF, hi = lo + G::TPF - 1, Kx = G::Kx, M = G::ROW_M;
        auto get = [&](int j, bool conj, bool zero_im) {
            const cd f = X[j * ld + ra], g = B_ROW ? X[j * ld + rb] : cd{0.0, 0.0};
            const double fy = zero_im ? 0.0 : f.y, gy = zero_im ? 0.0 : g.y;  // X_0 is read as real
            return conj ? cd{f.x + gy, g.x - fy} : cd{f.x - gy, fy + g.x};
        };
        if constexpr (hi <= Kx) {
            v[m] = get(lo + t, false, lo == 0 && t == 0);
        } else if constexpr (lo >= M - Kx) {
            v[m] = get(M - lo - t, true, false);
        } else if constexpr (lo > Kx && hi < M - Kx) {
            v[m] = cd{0.0, 0.0};
        } else {
            const int e = lo + t;
            const bool neg = lo >= M / 2, in = neg ? e >= M - Kx : e <= Kx;
            const cd x = get(in ? (neg ? M - e : e) : 0, neg, lo == 0 && t == 0);
            v[m] = in ? x : cd{0.0, 0.0};
        }
        row_gather_raw<G, B_ROW, m + 1>(X, ld, ra, rb, t, v);
    }
}

// Pass B forms u u_x as (1/2) (u^2)_x (two transforms per pair of rows) for rows of up to
// kSquareMaxM points, and as the product u * u_x (three transforms) for longer rows.
// Differentiating the square multiplies the round-off of mode j by q_j / 2, against the
// product's round-off of order |u u_x|: the ratio grows as Kx over the input's dominant mode
// index. Measured against the FP64 oracle on low-mode loops (|j| <= 8), the flow G of the
// square form errs by 1.1e-13 at 128 x 64, 4.9e-13 at 256 x 1024 and 3.8e-12 at 512 x 32
// (normwise), the product form by 1.7e-14, 3.0e-14 and 1.3e-13; with Kx <= 42 the square form
// stays inside the 1e-12 bound even for a loop made of its lowest mode.
constexpr int kSquareMaxM = 128;

// u u_x = (1/2) (u^2)_x on the rows of a pair: one inverse transform of u_a + i u_b, the squares
// (u_a^2) + i (u_b^2) in physical space and one forward transform (the factor i q_j / 2 is
// row_split's). Both fields are band-limited, so (u^2)_x of the band equals the band of 2 u u_x
// exactly; one transform of three is saved.
template <int M, int PT, bool XLOW, bool ALL>
__device__ __forceinline__ void row_square(cd* va, cd* ex, const TwCache<M, PT, ALL>& twc, const FftPos<M, PT, XLOW>& pos) {
    fft_inv<M, PT, XLOW>(va, ex, twc, pos);
#pragma unroll
    for (int m = 0; m < PT; ++m) va[m] = cd{va[m].x * va[m].x, va[m].y * va[m].y};
    fft_fwd<M, PT, XLOW>(va, ex, twc, pos);
}

// Products of two real fields f, g on the rows of a pair. The two inverse x-transforms take the
// rows of one field at a time (va = f_a + i f_b, vb = g_a + i g_b), so each transform carries
// values of one scale; packing f and g of one row together would let the round-off of the
// larger (r_x can exceed u by q_max^5) swamp the smaller. Then one forward transform of
// (f_a g_a) + i (f_b g_b).
template <int M, int PT, bool XLOW, bool ALL>
__device__ __forceinline__ void row_product(cd* va, cd* vb, cd* ex, const TwCache<M, PT, ALL>& twc,
                                            const FftPos<M, PT, XLOW>& pos) {
    fft_inv<M, PT, XLOW>(va, ex, twc, pos);
    fft_inv<M, PT, XLOW>(vb, ex, twc, pos);
#pragma unroll
    for (int m = 0; m < PT; ++m) va[m] = cd{va[m].x * vb[m].x, va[m].y * vb[m].y};
    fft_fwd<M, PT, XLOW>(va, ex, twc, pos);
}

// vb = i q va, the x-derivative of a pair's spectrum, q of the signed frequency e = t + m TPF
template <int M, int PT>
__device__ __forceinline__ void row_dx(const cd* va, int t, double dq, cd* vb) {
    constexpr int TPF = M / PT;
#pragma unroll
    for (int m = 0; m < PT; ++m) {
        const int e = t + m * TPF;
        const double q = dq * (double)((e <= M / 2) ? e : e - M);
        vb[m] = cd{-q * va[m].y, q * va[m].x};
    }
}

// The transforms of a block's pairs, between the staging barriers: the spectra of `fields`
// fields are staged in lds; on return the products' spectra are, and every thread may read
// them. Each wavefront's regions are its own until the barrier, so its exchanges reuse them.
// DX: the square form of u u_x (one field); otherwise the product of two fields, or of one field
// and its x-derivative.
template <int M, int PT, int FIELDS, int WR, bool DX, bool ALL>
__device__ __forceinline__ void row_transforms(const Shape& sh, cd* lds, const FftPos<M, PT>& pos,
                                               const TwCache<M, PT, ALL>& twc, cd* va, cd* vb) {
    using G = RowG<M, PT>;
    // the exchange addresses a wavefront's transforms as x * XS from the block's start: shift
    // the base so that they fall into the wavefront's own region
    const int wave = threadIdx.x / 64;
    cd* ex = lds + wave * (WR - G::PW * G::E::XS);
    if constexpr (DX)
        row_square<M, PT, false>(va, ex, twc, pos);
    else
        row_product<M, PT, false>(va, vb, ex, twc, pos);
    wave_lds_order();
    row_put<G>(lds + stage_base<G, WR>(pos.xs, 0), pos.t, va);
    __syncthreads();
}

// DMA copies raw tiles by the load unit (load_rows_lds, tiles of 64 rows or more) instead of
// staging packed spectra through registers. PT below the default spreads each row transform
// over more threads: tiles are then shorter, and a block covers the rows of one default-size
// tile (so that tile indices keep their meaning) in SUB consecutive sub-tiles.
template <int M, bool DMA = false, int PT = RowG<M>::PT>
__device__ __forceinline__ void row_pass_B(const Shape& sh, int block, const Work& w, cd* lds,
                                           const cd* __restrict__ tw) {
    using G = RowG<M, PT>;
    constexpr int SUB = RowG<M>::ROWS / G::ROWS;
    constexpr int WR = G::wave_region(1);
    constexpr bool DX = M <= kSquareMaxM;
    const size_t nrows = (size_t)sh.nloops * sh.N;
    const FftPos<M, PT> pos(threadIdx.x);
    TwCache<M, PT, kRowAll<M, PT>> twc;
    tw_cache_load<M, PT>(twc, pos, tw);
    auto sub = [&](size_t g0) {
        const cd* const src[1] = {w.A};
        cd va[PT], vb[PT];
        if constexpr (DMA) {
            load_rows_lds<G::ROWS, G::CMAX, G::TS, G::TILE, 1>(lds, src, g0, sh, nrows);
            __syncthreads();
            row_gather_raw<G, true>(lds, G::TS, pos.xs, G::P + pos.xs, pos.t, va);
            __syncthreads();  // every wavefront has read the tile: its regions are free
        } else {
            RowLoad<G, 1> ld;
            ld.issue(src, g0, sh, nrows);
            ld.template commit<WR>(lds);
            __syncthreads();
            row_gather<G>(lds + stage_base<G, WR>(pos.xs, 0), pos.t, va);
            wave_lds_order();
        }
        if constexpr (!DX) row_dx<M, PT>(va, pos.t, kTwoPi / sh.L, vb);
        row_transforms<M, PT, 1, WR, DX>(sh, lds, pos, twc, va, vb);
        row_store<G, WR, DX>(lds, w.BD, g0, sh, nrows);
    };
    const size_t gb = (size_t)block * RowG<M>::ROWS;
    if constexpr (SUB == 1) {
        sub(gb);
    } else {
#pragma unroll 1
        for (int h = 0; h < SUB; ++h) {
            if (h > 0) __syncthreads();  // the previous sub-tile's rows have been read
            sub(gb + (size_t)h * G::ROWS);
        }
    }
}

// Sum the per-column partials of loop l into J, dJ/dT; in MODE_STEP also advance T.
// Called by all 64 lanes of one wavefront: lanes add strided partials in a fixed order, then
// an xor tree combines them.
__device__ __forceinline__ void finalize_loop(const Shape& sh, int l, const Work& w, double* T, int mode,
                                              double dtau, double* J_hist, double* Jout, double* dJdTout) {
    const int lane = threadIdx.x % 64;
    const double* pp = w.partial + (size_t)l * sh.C * 2;
    double sj = 0.0, st = 0.0;
    for (int j = lane; j < sh.C; j += 64) {
        sj += pp[2 * j];
        st += pp[2 * j + 1];
    }
    sj = sum_lanes<32>(sj);
    st = sum_lanes<32>(st);
    if (lane != 0) return;
    const double Tl = T[l];
    const double J = 0.5 * sh.L * sj;
    const double dJdT = sh.L * st / (Tl * Tl);
    w.J[l] = J;
    w.dJdT[l] = dJdT;
    if (Jout) Jout[l] = J;
    if (dJdTout) dJdTout[l] = dJdT;
    bool bad = !(Tl > 0.0) || !isfinite(Tl) || !isfinite(J) || !isfinite(dJdT);
    if (mode == MODE_STEP) {
        const double Tn = Tl - dtau * dJdT;
        w.Told[l] = Tl;
        T[l] = Tn;
        if (J_hist) J_hist[l] = J;
        bad = bad || !(Tn > 0.0) || !isfinite(Tn);
    }
    if (bad) atomicCAS(w.status, 0, -4);
}

template <int M, bool DMA = false, int PT = RowG<M>::PT>
__device__ __forceinline__ void row_pass_D(const Shape& sh, int block, const Work& w, double* T, int mode,
                                           double dtau, double* J_hist, double* Jout, double* dJdTout, cd* lds,
                                           const cd* __restrict__ tw) {
    using G = RowG<M, PT>;
    constexpr int SUB = RowG<M>::ROWS / G::ROWS;
    const size_t nrows = (size_t)sh.nloops * sh.N;
    const size_t gb = (size_t)block * RowG<M>::ROWS;
    // Loops whose first row lies in this block are finished here (partials from pass C), by
    // wavefront 0 while the first sub-tile's loads are in flight.
    auto finalize = [&]() {
        if (mode != MODE_ADJOINT && threadIdx.x < 64) {
            const size_t l0 = (gb + sh.N - 1) >> sh.logN;  // first loop starting at or after gb
            for (size_t l = l0; (l << sh.logN) < gb + RowG<M>::ROWS && l < (size_t)sh.nloops; ++l)
                finalize_loop(sh, (int)l, w, T, mode, dtau, J_hist, Jout, dJdTout);
        }
    };
    constexpr int WR = G::wave_region(2);
    const FftPos<M, PT> pos(threadIdx.x);
    TwCache<M, PT, kRowAll<M, PT>> twc;
    tw_cache_load<M, PT>(twc, pos, tw);
    auto sub = [&](size_t g0, bool first) {
        const cd* const src[2] = {w.A, w.Cb};
        cd va[PT], vb[PT];  // u and r_x
        if constexpr (DMA) {
            load_rows_lds<G::ROWS, G::CMAX, G::TS, G::TILE, 2, false>(lds, src, g0, sh, nrows);
            if (first) finalize();
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            row_gather_raw<G, true>(lds, G::TS, pos.xs, G::P + pos.xs, pos.t, va);
            row_gather_raw<G, true>(lds + G::TILE, G::TS, pos.xs, G::P + pos.xs, pos.t, vb);
            __syncthreads();  // every wavefront has read the tiles: its regions are free
        } else {
            RowLoad<G, 2> ld;
            ld.issue(src, g0, sh, nrows);
            if (first) finalize();
            ld.template commit<WR>(lds);
            __syncthreads();
            row_gather<G>(lds + stage_base<G, WR>(pos.xs, 0), pos.t, va);
            row_gather<G>(lds + stage_base<G, WR>(pos.xs, 1), pos.t, vb);
            wave_lds_order();
        }
        row_transforms<M, PT, 2, WR, false>(sh, lds, pos, twc, va, vb);
        row_store<G, WR, false>(lds, w.BD, g0, sh, nrows);
    };
    if constexpr (SUB == 1) {
        sub(gb, true);
    } else {
#pragma unroll 1
        for (int h = 0; h < SUB; ++h) {
            if (h > 0) __syncthreads();  // the previous sub-tile's rows have been read
            sub(gb + (size_t)h * G::ROWS, h == 0);
        }
    }
}

}  // namespace lo
