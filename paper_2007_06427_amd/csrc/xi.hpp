// Centre-symmetric loops (Sec. 3, eq. KS_loop_sym): a loop with u(-x, s) = -u(x, s) for every
// s is invariant under Xi, and the flow keeps it so. Every field of the step then has a fixed
// parity in x: u, u u_x, r and u r_x are odd, u_x and r_x even. An odd real field has a
// purely imaginary x-spectrum at every s (column j = 0 vanishes) and an even one a real
// x-spectrum, so one real number per (j, s) carries a column, and in s each column is the
// transform of a real sequence (Hermitian in k). State and intermediates halve.
//
// Per loop, with Kx the band edge in j and K1 = Ks + 1:
//   U, G  [j-1][k], j = 1..Kx, k = 0..Ks (complex): b_{j,k} = -i u_hat_{j,k}, Hermitian in k
//         (b_{j,-k} = conj b_{j,k}, b_{j,0} real); G holds U1 = b + dtau sigma G_lin;
//   A     [j-1][n] (real): Im u_j(s_n);    B then D: Im (u u_x)_j, Im (u r_x)_j;
//   C     [j-1][n] (real): (r_x)_j(s_n), which is real.
// In terms of b the residual, cost, period derivative and update take the forms of the full
// path (each term is linear in u_hat, so the factor -i passes through); the sums over the
// band run over j >= 1 (w_j = 2) and k >= 0, with k > 0 counted twice.
//
// Column transforms carry two columns j = 2c + 1, 2c + 2 in one complex transform
// (z = b_{2c+1}(s) + i b_{2c+2}(s)); row transforms are those of the full path on the odd and
// even half spectra.
#pragma once

#include "passes.hpp"

namespace lo {

struct XiWork {
    cd* U;
    cd* G;
    double* A;
    double* BD;
    double* Cb;
    double* partial;  // [l][j-1][2]
    double* J;
    double* dJdT;
    double* Told;
    int* status;
};

// ----------------------------------------------------------------------------- columns
// The column pairs of a thread: spectrum side (l, j1, t, two), points side (active_t, two_t, col_t).
template <int N>
struct XiColPos {
    using G = ColG<N>;
    FftPos<N, G::PT> p;
    bool active, two;  // two: the pair's second column exists (Kx may be odd)
    int l, j1, t;      // j1: 0-based index (j - 1) of the pair's first column
    bool active_t, two_t;
    size_t col_t;      // index l Kx + j1 of the points side's pair
    __device__ __forceinline__ XiColPos(const Shape& sh, int block) : p(threadIdx.x) {
        const int NP = (sh.Kx + 1) / 2, n = sh.nloops * NP;
        const int gc = block * G::F + p.xs, gt = block * G::F + p.xt;
        t = p.t;
        active = gc < n;
        l = active ? gc / NP : 0;
        j1 = active ? 2 * (gc % NP) : 0;
        two = active && j1 + 1 < sh.Kx;
        active_t = gt < n;
        const int jt = active_t ? 2 * (gt % NP) : 0;
        two_t = active_t && jt + 1 < sh.Kx;
        col_t = active_t ? (size_t)(gt / NP) * sh.Kx + jt : 0;
    }
};

// Spectrum element e (FFT order) of z = b1 + i b2 from the half spectra c1 = b1_hat, c2 =
// b2_hat (k = 0..Ks) through Hermitian symmetry.
__device__ __forceinline__ cd xi_pack(const cd* c1, const cd* c2, int e, int N, int Ks, bool two) {
    if (e <= Ks) {
        const cd x = c1[e], y = two ? c2[e] : cd{0.0, 0.0};
        return cd{x.x - y.y, x.y + y.x};
    }
    if (e >= N - Ks) {
        const cd x = c1[N - e], y = two ? c2[N - e] : cd{0.0, 0.0};
        return cd{x.x + y.y, y.x - x.y};  // conj(x) + i conj(y)
    }
    return cd{0.0, 0.0};
}

// After a forward transform of z = b1 + i b2 (values v, thread t holding e = t + m TPF):
// the half spectra of b1 and b2, scaled by s, through the exchange region ex:
// b1_hat(e) = (Z_e + conj Z_{N-e}) / 2, b2_hat(e) = (Z_e - conj Z_{N-e}) / (2 i).
template <int N>
__device__ __forceinline__ void xi_split(const cd* v, int t, cd* ex, double s, cd* p1, cd* p2) {
    using G = ColG<N>;
    xsync<G::TPF>();  // the transform's other wavefront may still read its part of the region
#pragma unroll
    for (int m = 0; m < G::PT; ++m) ex[t + m * G::TPF] = v[m];
    xsync<G::TPF>();
#pragma unroll
    for (int m = 0; m < G::PT; ++m) {
        const int e = t + m * G::TPF;
        const cd w = ex[(N - e) & (N - 1)];
        const cd z = v[m];
        p1[m] = cd{0.5 * s * (z.x + w.x), 0.5 * s * (z.y - w.y)};
        p2[m] = cd{0.5 * s * (z.y + w.y), 0.5 * s * (w.x - z.x)};
    }
    xsync<G::TPF>();
}

// Hermitian extension in k of two half spectra held in registers (element e of g1, g2 at
// k = e <= Ks), through ex, into the inverse-transform input of z = b1 + i b2.
template <int N>
__device__ __forceinline__ void xi_extend(cd* v, const cd* g1, const cd* g2, int t, int Ks, bool two, cd* ex) {
    using G = ColG<N>;
#pragma unroll
    for (int m = 0; m < G::PT; ++m) {
        const int e = t + m * G::TPF;
        if (e <= Ks) {
            ex[e] = g1[m];
            ex[e + Ks + 1] = g2[m];
        }
    }
    xsync<G::TPF>();
#pragma unroll
    for (int m = 0; m < G::PT; ++m) {
        const int e = t + m * G::TPF;
        cd z{0.0, 0.0};
        if (e <= Ks || e >= N - Ks) {
            const int k = e <= Ks ? e : N - e;
            const cd x = ex[k], y = two ? ex[k + Ks + 1] : cd{0.0, 0.0};
            z = e <= Ks ? cd{x.x - y.y, x.y + y.x} : cd{x.x + y.y, y.x - x.y};
        }
        v[m] = z;
    }
    xsync<G::TPF>();
}

template <int N>
__device__ __forceinline__ void xi_store_pair(const XiColPos<N>& p, const cd* v, double* X) {
    using G = ColG<N>;
    if (!p.active_t) return;
    double* x1 = X + p.col_t * N;
#pragma unroll
    for (int m = 0; m < G::PT; ++m) {
        const int n = p.p.point(m);
        x1[n] = v[m].x;
        if (p.two_t) x1[N + n] = v[m].y;
    }
}

template <int N>
__device__ __forceinline__ void xi_load_pair(const XiColPos<N>& p, const double* X, cd* v) {
    using G = ColG<N>;
    const double* x1 = X + p.col_t * N;
#pragma unroll
    for (int m = 0; m < G::PT; ++m) {
        const int n = p.p.point(m);
        v[m] = p.active_t ? cd{x1[n], p.two_t ? x1[N + n] : 0.0} : cd{0.0, 0.0};
    }
}

// Pass A: the inverse s-transforms of a pair of band columns into A.
template <int N>
__device__ __forceinline__ void xi_col_pass_A(const Shape& sh, int block, const XiWork& w, cd* ex,
                                              const cd* __restrict__ tw) {
    using G = ColG<N>;
    const XiColPos<N> p(sh, block);
    TwCache<N, G::PT> twc;
    tw_cache_load<N, G::PT>(twc, p.p, tw);
    const int K1 = sh.Ks + 1;
    const cd* b1 = w.U + ((size_t)p.l * sh.Kx + p.j1) * K1;
    cd v[G::PT];
#pragma unroll
    for (int m = 0; m < G::PT; ++m)
        v[m] = p.active ? xi_pack(b1, b1 + K1, p.t + m * G::TPF, N, sh.Ks, p.two) : cd{0.0, 0.0};
    fft_inv<N, G::PT>(v, ex, twc, p.p);
    xi_store_pair<N>(p, v, w.A);
}

// Pass C: residual, the partial sums of J and dJ/dT, U1, and the inverse transform of r_x.
template <int N>
__device__ __forceinline__ void xi_col_pass_C(const Shape& sh, int block, const double* __restrict__ T,
                                              const XiWork& w, double dtau, int scheme, cd* ex, double* red,
                                              const cd* __restrict__ tw) {
    using G = ColG<N>;
    const XiColPos<N> p(sh, block);
    cd* exf = ex + p.p.xs * Fft<N, G::PT>::XS;  // the spectrum side's region, for split and extension
    TwCache<N, G::PT> twc;
    tw_cache_load<N, G::PT>(twc, p.p, tw);
    cd v[G::PT];
    xi_load_pair<N>(p, w.BD, v);
    fft_fwd<N, G::PT>(v, ex, twc, p.p);
    cd p1[G::PT], p2[G::PT];
    xi_split<N>(v, p.t, exf, 1.0 / N, p1, p2);

    const double invT = 1.0 / (p.active ? T[p.l] : 1.0);
    const int K1 = sh.Ks + 1;
    const ColCoef f[2] = {ColCoef(p.j1 + 1, sh.L), ColCoef(p.j1 + 2, sh.L)};
    double Jp[2] = {0.0, 0.0}, dTp[2] = {0.0, 0.0};
    cd g1[G::PT], g2[G::PT];
    static_for<G::PT>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        using B = BandSlot<N, m>;
        g1[m] = cd{0.0, 0.0};
        g2[m] = cd{0.0, 0.0};
        if (B::neg || !p.active || !B::in(p.t)) return;  // k = 0 .. Ks
        const int e = p.t + m * G::TPF;
        const double om = kTwoPi * e;
        const double a = om * invT;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (c == 1 && !p.two) break;
            const size_t at = ((size_t)p.l * sh.Kx + p.j1 + c) * K1 + e;
            const cd b = w.U[at];
            // the residual, sums and update in the b form; w_j = 2 (j >= 1), k > 0 counted twice
            const cd r = band_residual(f[c], a, 1.0, b, c == 0 ? p1[m] : p2[m]);
            double j = 0.0, t = 0.0;
            band_sums(om, b, r, j, t);
            const double wk = (e == 0) ? 2.0 : 4.0;
            Jp[c] = __builtin_fma(wk, j, Jp[c]);
            dTp[c] = __builtin_fma(wk, t, dTp[c]);
            const cd gl = band_glin(f[c], a, r);
            const double st = band_step(f[c], a, dtau, scheme);
            w.G[at] = cd{__builtin_fma(st, gl.x, b.x), __builtin_fma(st, gl.y, b.y)};  // U1
            const cd rx = cd{-f[c].q * r.x, -f[c].q * r.y};  // (r_x)_hat in the real-column form
            if (c == 0)
                g1[m] = rx;
            else
                g2[m] = rx;
        }
    });
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        double jp = Jp[c], tp = dTp[c];
        col_sum2<N>(jp, tp, red);
        if (p.active && p.t == 0 && (c == 0 || p.two)) {
            double* part = w.partial + ((size_t)p.l * sh.Kx + p.j1 + c) * 2;
            part[0] = jp;
            part[1] = tp;
        }
    }
    xi_extend<N>(v, g1, g2, p.t, sh.Ks, p.two, exf);
    fft_inv<N, G::PT>(v, ex, twc, p.p);
    xi_store_pair<N>(p, v, w.Cb);
}

// Pass E: the new state U1 - dtau sigma (u r_x)_hat, then the next step's A from it.
template <int N>
__device__ __forceinline__ void xi_col_pass_E(const Shape& sh, int block, const XiWork& w, double dtau, int scheme,
                                              bool fuseA, cd* ex, const cd* __restrict__ tw) {
    using G = ColG<N>;
    const XiColPos<N> p(sh, block);
    cd* exf = ex + p.p.xs * Fft<N, G::PT>::XS;  // the spectrum side's region, for split and extension
    TwCache<N, G::PT> twc;
    tw_cache_load<N, G::PT>(twc, p.p, tw);
    cd v[G::PT];
    xi_load_pair<N>(p, w.BD, v);
    fft_fwd<N, G::PT>(v, ex, twc, p.p);
    cd p1[G::PT], p2[G::PT];
    xi_split<N>(v, p.t, exf, 1.0 / N, p1, p2);
    const double invT = 1.0 / (p.active ? w.Told[p.l] : 1.0);
    const int K1 = sh.Ks + 1;
    const ColCoef f[2] = {ColCoef(p.j1 + 1, sh.L), ColCoef(p.j1 + 2, sh.L)};
    cd g1[G::PT], g2[G::PT];
    static_for<G::PT>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        using B = BandSlot<N, m>;
        g1[m] = cd{0.0, 0.0};
        g2[m] = cd{0.0, 0.0};
        if (B::neg || !p.active || !B::in(p.t)) return;
        const int e = p.t + m * G::TPF;
        const double a = kTwoPi * e * invT;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (c == 1 && !p.two) break;
            const size_t at = ((size_t)p.l * sh.Kx + p.j1 + c) * K1 + e;
            const cd x = band_update(w.G[at], c == 0 ? p1[m] : p2[m], band_step(f[c], a, dtau, scheme));
            w.U[at] = x;
            if (c == 0)
                g1[m] = x;
            else
                g2[m] = x;
        }
    });
    if (!fuseA) return;
    xi_extend<N>(v, g1, g2, p.t, sh.Ks, p.two, exf);
    fft_inv<N, G::PT>(v, ex, twc, p.p);
    xi_store_pair<N>(p, v, w.A);
}

// -------------------------------------------------------------------------------- rows
// The rows of NT real intermediates for this thread's items (RowLoad for real columns j = 1..Kx):
// field 0 is odd in x (spectrum i f_j), field 1 even (f_j); their packed spectra are staged.
template <class G, int NT>
struct XiRowLoad {
    double fa[NT][G::NL], fb[NT][G::NL];
    __device__ __forceinline__ void issue(const double* const (&X)[NT], size_t g0, const Shape& sh, size_t nrows) {
#pragma unroll
        for (int k = 0; k < G::NL; ++k) {
            int p, j;
            const bool item = row_item<G>(k, p, j) && j > 0;
            const size_t ga = g0 + p, gb = ga + G::P;
            const bool oka = item && ga < nrows, okb = item && gb < nrows;
            const size_t a = oka ? xi_row_offset(ga, j, sh) : 0, b = okb ? xi_row_offset(gb, j, sh) : 0;
#pragma unroll
            for (int q = 0; q < NT; ++q) {
                fa[q][k] = oka ? X[q][a] : 0.0;
                fb[q][k] = okb ? X[q][b] : 0.0;
            }
        }
    }
    static __device__ __forceinline__ size_t xi_row_offset(size_t g, int j, const Shape& sh) {
        return ((g >> sh.logN) * sh.Kx + (j - 1)) * sh.N + (g & (size_t)(sh.N - 1));
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
                const double f = fa[q][k], g = fb[q][k];  // zero for j = 0: that column vanishes
                const int neg = j == 0 ? 0 : G::ROW_M - G::SH - j;
                if (q == 0) {
                    z[neg] = cd{g, -f};
                    z[j] = cd{-g, f};
                } else {
                    z[neg] = cd{f, g};
                    z[j] = cd{f, g};
                }
            }
        }
    }
};

// The imaginary parts of the rows' half spectra (an odd product: its real parts vanish) for
// j = 1..Kx, from the staged products, into the real intermediate X.
template <class G, int WR>
__device__ __forceinline__ void xi_row_store(const cd* lds, double* X, size_t g0, const Shape& sh, size_t nrows) {
    constexpr double s = 0.5 / G::ROW_M;
#pragma unroll
    for (int k = 0; k < G::NL; ++k) {
        int p, j;
        if (!row_item<G>(k, p, j) || j == 0) continue;
        const cd* z = lds + stage_base<G, WR>(p, 0);
        const cd a = z[j], b = z[G::ROW_M - G::SH - j];
        const size_t ga = g0 + p, gb = ga + G::P;
        if (ga < nrows) X[XiRowLoad<G, 1>::xi_row_offset(ga, j, sh)] = (a.y - b.y) * s;
        if (gb < nrows) X[XiRowLoad<G, 1>::xi_row_offset(gb, j, sh)] = (b.x - a.x) * s;
    }
}

template <int M>
__device__ __forceinline__ void xi_row_pass_B(const Shape& sh, int block, const XiWork& w, cd* lds,
                                              const cd* __restrict__ tw) {
    using G = RowG<M>;
    constexpr int WR = G::wave_region(1);
    const size_t nrows = (size_t)sh.nloops * sh.N;
    const size_t g0 = (size_t)block * G::ROWS;
    const FftPos<M, G::PT> pos(threadIdx.x);
    TwCache<M, G::PT, kRowAll<M>> twc;
    tw_cache_load<M, G::PT>(twc, pos, tw);
    const double* const src[1] = {w.A};
    XiRowLoad<G, 1> ld;
    ld.issue(src, g0, sh, nrows);
    ld.template commit<WR>(lds);
    __syncthreads();
    cd va[G::PT], vb[G::PT];
    row_gather<G>(lds + stage_base<G, WR>(pos.xs, 0), pos.t, va);
    wave_lds_order();
    row_dx<M, G::PT>(va, pos.t, kTwoPi / sh.L, vb);
    row_transforms<M, G::PT, 1, WR, false>(sh, lds, pos, twc, va, vb);
    xi_row_store<G, WR>(lds, w.BD, g0, sh, nrows);
}

template <int M>
__device__ __forceinline__ void xi_row_pass_D(const Shape& sh, int block, const XiWork& w, double* T,
                                              double dtau, double* J_hist, cd* lds, const cd* __restrict__ tw) {
    using G = RowG<M>;
    constexpr int WR = G::wave_region(2);
    const size_t nrows = (size_t)sh.nloops * sh.N;
    const size_t g0 = (size_t)block * G::ROWS;
    const FftPos<M, G::PT> pos(threadIdx.x);
    TwCache<M, G::PT, kRowAll<M>> twc;
    tw_cache_load<M, G::PT>(twc, pos, tw);
    const double* const src[2] = {w.A, w.Cb};
    XiRowLoad<G, 2> ld;
    ld.issue(src, g0, sh, nrows);
    // loops whose first row lies in this block are finished here (partials from pass C)
    if (threadIdx.x < 64) {
        Shape sx = sh;
        sx.C = sh.Kx;  // one partial pair per column j = 1..Kx
        Work wf{};
        wf.partial = w.partial;
        wf.J = w.J;
        wf.dJdT = w.dJdT;
        wf.Told = w.Told;
        wf.status = w.status;
        const size_t l0 = (g0 + sh.N - 1) >> sh.logN;
        for (size_t l = l0; (l << sh.logN) < g0 + G::ROWS && l < (size_t)sh.nloops; ++l)
            finalize_loop(sx, (int)l, wf, T, MODE_STEP, dtau, J_hist, nullptr, nullptr);
    }
    ld.template commit<WR>(lds);
    __syncthreads();
    cd va[G::PT], vb[G::PT];
    row_gather<G>(lds + stage_base<G, WR>(pos.xs, 0), pos.t, va);
    row_gather<G>(lds + stage_base<G, WR>(pos.xs, 1), pos.t, vb);
    wave_lds_order();
    row_transforms<M, G::PT, 2, WR, false>(sh, lds, pos, twc, va, vb);
    xi_row_store<G, WR>(lds, w.BD, g0, sh, nrows);
}

}  // namespace lo
