// LDS-resident form of the fictitious-time step (Sec. 4.2): one block runs every pass of every
// step of one loop in one launch, so HBM sees only the state's load and store. It applies where
// a loop's two live intermediates fit in the 160 KB of LDS of a CU (for example 32 x 256,
// 64 x 128, 128 x 64).
//
// The passes are those of passes.hpp with the same row pairs, transforms, band functions and
// fixed-order sums, so a step gives the same bits as the HBM form; what differs is where values
// live. A thread keeps the same column and the same pair of rows for the whole launch, so
// everything that a pass hands to a later pass of the same thread stays in registers:
//   the band state u of its column (pass C turns it into U1, pass E into the new state),
//   dtau sigma of its modes, from pass C to pass E,
//   u on the grid of its row pair, from pass B to pass D (whose own transform would only repeat it),
//   the twiddles of both transforms.
// Only what changes hands between threads goes through LDS (complex values unless noted), for a
// loop of M x N (Nx x Ns):
//   A  [C][N+1]  u after the inverse s-transforms (pass A, or E fused with the next A)
//   X  [C][N+1]  B, then C (in place, column by column), then D (in place, pair by pair)
//   EX           exchange regions of the transforms, and the pairs' products before their split
//   2C doubles   per-column partial sums of J and dJ/dT
//   4 doubles    T, T_old, J, dJ/dT
// Columns of A and X are N + 1 apart: a row pass reads 16 columns of a row, or a short column
// pass a point of 16 columns, at a time, and the odd stride puts them on different banks.
//
// What bounds it is instruction issue and LDS latency in the few wavefronts of a loop: the block
// has just the threads that one round of every pass needs (64 to 512), and wavefronts that have
// no rows or no columns skip that pass's transforms. With the state in LDS, u transformed twice,
// every pass loading its twiddles and blocks of 256 threads for every shape, a step of one 32 x 32
// loop took 6.6 us (now 4.6), of 256 loops of 64 x 64 12.2 (7.4), of one 64 x 128 loop 25 (12.9; the
// per-pass form 19).
#pragma once

#include "passes.hpp"

namespace lo {

template <int M, int N>
struct ResG {
    using R = RowG<M>;
    static constexpr int PT = 8;
    static constexpr int C = (M - 1) / 3 + 1;
    static constexpr int Ks = (N - 1) / 3;
    static constexpr int NB = 2 * Ks + 1;
    static constexpr int H = M / 2 + 1;
    static constexpr int LD = N + 1;
    static constexpr int W = C * LD;
    // Rows are paired as the HBM form's tiles pair the rows of one loop: (a, a + P); a loop of
    // at most P rows leaves the second row of every pair empty.
    static constexpr int P = R::P;
    static constexpr bool B_ROW = N >= 2 * P;
    static constexpr int PAIRS = B_ROW ? N / 2 : N;
    static constexpr int NEED = PAIRS * R::TPF > C * (N / PT) ? PAIRS * R::TPF : C * (N / PT);
    static constexpr int NT = NEED <= 64 ? 64 : NEED <= 128 ? 128 : NEED <= 256 ? 256 : 512;
    using RF = Fft<M, PT, true>;  // row lanes are pair-fastest: consecutive lanes on consecutive rows
    using CF = Fft<N, PT>;
    static constexpr int ZS = RF::L == 1 ? 2 * R::Kx + 1 : RF::XS;  // region of a pair
    // exchange space of the first `waves` wavefronts, in the row and the column passes
    static constexpr int CW = (C + CF::XPW - 1) / CF::XPW;  // wavefronts with columns
    static constexpr int rx(int waves) { return waves * RF::XPW * ZS; }
    static constexpr int cx(int waves) { return CF::L == 1 ? 0 : (waves < CW ? waves : CW) * CF::XPW * CF::XS; }
    static constexpr int ex(int waves) { return rx(waves) > cx(waves) ? rx(waves) : cx(waves); }
    // SPLIT (64 x 128 and 128 x 64): the exchange space of all eight wavefronts does not fit beside A
    // and X. Wavefronts 4 .. 7 then use whichever of A and X holds nothing in that pass: X in
    // passes B and E (two more barriers per step: before B writes X, and after E has read it),
    // A in passes C and D.
    static constexpr int DOUBLES = 2 * C + 4;
    static constexpr size_t bytes(int e) { return sizeof(cd) * (size_t)(2 * W + e) + sizeof(double) * DOUBLES; }
    static constexpr bool SPLIT = NT == 512 && bytes(ex(8)) > 160 * 1024;
    static constexpr int EX = ex(SPLIT ? 4 : NT / 64);
    static constexpr size_t BYTES = bytes(EX);
    static constexpr bool FITS = BYTES <= 160 * 1024 && N <= 512 && M <= 128 && NEED <= 512 &&
                                 (!SPLIT || PAIRS * R::TPF == NT);  // every wavefront reaches its barriers
    // Twiddle powers kept in registers (TwCache) where they fit: 16 registers for each stage that
    // has twiddles. Kept for rows and columns, for one of them, or (SPLIT 64 x 128) for neither;
    // a step forms 4 or 8 products less per transform (a step of one 32 x 32 loop 4.93 -> 4.61 us,
    // of 256 of 64 x 64 7.7 -> 7.4; 64 x 128, where they spill, would go from 12.9 to 14.1).
    static constexpr int TW_M = 16 * (RF::L - (RF::F == 1)), TW_N = 16 * (CF::L - (CF::F == 1));
    static constexpr bool TW_BOTH = NT <= 128 || TW_M + TW_N <= 32;
    static constexpr bool TW_ROWS = TW_BOTH || (TW_M == 16 && !SPLIT);
    static constexpr bool TW_COLS = TW_BOTH || (TW_M == 32 && TW_N == 16);
    // Wavefronts per SIMD the kernel is compiled for: two (at most 256 registers each), so that
    // blocks of small loops share a CU, except where LDS holds one block of four wavefronts.
    static constexpr int WPE = NT == 256 && BYTES > 80 * 1024 ? 1 : 2;
};

// Split of the products' spectrum (slots va) into rows a and b of X, through the pair's region z.
// SYNC: z lies in X, so the block waits for every wavefront to have read its part.
template <int M, int N, bool DX, bool SYNC>
__device__ __forceinline__ void res_split(double L, const cd* va, cd* z, int t, cd* X, int a, bool on) {
    using R = ResG<M, N>;
    using G = RowG<M>;
    constexpr int NJ = (G::CMAX + G::TPF - 1) / G::TPF;
    row_put<G>(z, t, va);
    wave_lds_order();
    cd wa[NJ], wb[NJ];
#pragma unroll
    for (int i = 0; i < NJ; ++i) {
        const int j = t + i * G::TPF < G::CMAX ? t + i * G::TPF : 0;
        row_split<M, DX>(L, j, z[j], z[j == 0 ? 0 : M - G::SH - j], wa[i], wb[i]);
    }
    if constexpr (SYNC)
        __syncthreads();
    else
        wave_lds_order();  // the region is reused by this group's next transform
    if (!on) return;
#pragma unroll
    for (int i = 0; i < NJ; ++i) {
        const int j = t + i * G::TPF;
        if (j < G::CMAX) {
            X[j * R::LD + a] = wa[i];
            if (R::B_ROW) X[j * R::LD + a + R::P] = wb[i];
        }
    }
}

// All of a block's work for one loop: nsteps steps (src -> dst in the rfft layout, *T in place, J of
// step i into J_hist[i * jstride]), or, with GRAD, the flow G_1 into dst and J, dJ/dT into *Jout,
// *dJdTout. J_hist, Jout and dJdTout may be null; src and dst may be the same.
template <int M, int N, bool GRAD>
__device__ __forceinline__ void resident_loop(double L, const cd* src, cd* dst, double* T, double dtau, int scheme,
                                              int nsteps, double* J_hist, int jstride, double* Jout, double* dJdTout,
                                              int* status, cd* lds, const cd* __restrict__ tw) {
    using R = ResG<M, N>;
    using G = RowG<M>;
    constexpr int PT = R::PT, LD = R::LD;
    static_assert(!R::SPLIT || (R::rx(8) - R::rx(4) <= R::W && R::cx(8) - R::cx(4) <= R::W), "A and X hold the split");
    cd* A = lds;
    cd* X = A + R::W;
    cd* EX = X + R::W;
    double* part = reinterpret_cast<double*>(EX + R::EX);
    double* sc = part + 2 * R::C;  // T, T_old, J, dJ/dT
    const int tid = threadIdx.x, wave = tid / 64;
    const FftPos<M, PT, true> pr(tid);
    const FftPos<N, PT> pc(tid);
    // this thread's rows a and a + P, its column j (spectrum side) and jt (points side)
    const bool row_on = pr.xs < R::PAIRS;
    const int a = row_on ? pr.xs / R::P * 2 * R::P + pr.xs % R::P : 0;
    const bool rows_here = wave * R::RF::XPW < R::PAIRS;  // this wavefront has rows, has columns
    const bool cols_here = wave * R::CF::XPW < R::C;
    const int j = pc.xs;
    const bool col_on = j < R::C, pts_on = pc.xt < R::C;
    cd* const acol = A + (pts_on ? pc.xt : 0) * LD;
    cd* const xcol = X + (pts_on ? pc.xt : 0) * LD;
    // exchange spaces of this wavefront in passes B and D, C and E (addressed as x XS, x the
    // transform's index in the block)
    const bool alt = R::SPLIT && wave >= 4;
    cd* const exB = alt ? X - R::rx(4) : EX;
    cd* const exD = alt ? A - R::rx(4) : EX;
    cd* const exC = alt ? A - R::cx(4) : EX;
    cd* const exE = alt ? X - R::cx(4) : EX;
    TwCache<M, PT, R::TW_ROWS> twr;
    TwCache<N, PT, R::TW_COLS> twc;
    tw_cache_load<M, PT>(twr, pr, tw);
    tw_cache_load<N, PT>(twc, pc, tw);
    const ColCoef f(col_on ? j : 0, L);
    const double wj = (j == 0) ? 1.0 : 2.0;
    constexpr double invN = 1.0 / N;
    Work w{};
    w.partial = part;
    w.J = sc + 2;
    w.dJdT = sc + 3;
    w.Told = sc + 1;
    w.status = status;
    Shape s1{};
    s1.C = R::C;
    s1.N = N;
    s1.L = L;
    s1.nloops = 1;

    cd u[PT], ug[PT], v[PT];
    double s[PT];
    static_for<PT>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        using B = BandSlot<N, m>;
        cd x{0.0, 0.0};
        s[m] = 0.0;
        ug[m] = cd{0.0, 0.0};
        if (col_on && B::in(pc.t)) {
            const int e = pc.t + m * B::TPF;
            x = src[(size_t)e * R::H + j];
            if (j == 0) {
                const cd q = src[(size_t)((N - e) & (N - 1)) * R::H];
                x = cd{0.5 * (x.x + q.x), 0.5 * (x.y - q.y)};
            }
        }
        u[m] = x;
    });
    if (tid == 0) sc[0] = *T;
    auto store_col = [&](cd* col) {  // v (points) into a column of A or X
        if (pts_on)
#pragma unroll
            for (int m = 0; m < PT; ++m) col[pc.point(m)] = v[m];
    };
    auto load_col = [&]() {
#pragma unroll
        for (int m = 0; m < PT; ++m) v[m] = pts_on ? xcol[pc.point(m)] : cd{0.0, 0.0};
    };
    auto inverse_u = [&]() {  // pass A
#pragma unroll
        for (int m = 0; m < PT; ++m) v[m] = u[m];
        fft_inv<N, PT>(v, exE, twc, pc);
        store_col(acol);
    };
    if (nsteps > 0 && cols_here) inverse_u();
    __syncthreads();
#pragma unroll 1
    for (int st = 0; st < nsteps; ++st) {
        if (rows_here) {  // pass B: (1/2) (u^2)_x (with SPLIT every wavefront has rows)
            static_assert(M <= kSquareMaxM, "the resident form takes the square form of u u_x");
            row_gather_raw<G, R::B_ROW>(A, LD, a, a + R::P, pr.t, ug);
            fft_inv<M, PT, true>(ug, exB, twr, pr);
#pragma unroll
            for (int m = 0; m < PT; ++m) v[m] = cd{ug[m].x * ug[m].x, ug[m].y * ug[m].y};
            fft_fwd<M, PT, true>(v, exB, twr, pr);
            res_split<M, N, true, R::SPLIT>(L, v, exB + pr.xs * R::ZS, pr.t, X, a, row_on);
        }
        __syncthreads();
        const double invT = 1.0 / sc[0];
        if (cols_here) {  // pass C
            load_col();
            fft_fwd<N, PT>(v, exC, twc, pc);
            double Jp = 0.0, dTp = 0.0;
            static_for<PT>([&](auto mc) {
                constexpr int m = decltype(mc)::value;
                using B = BandSlot<N, m>;
                cd x{0.0, 0.0};
                if (col_on && B::in(pc.t)) {
                    const double om = kTwoPi * B::k(pc.t), ak = om * invT;
                    const cd r = band_residual(f, ak, invN, u[m], v[m]);
                    band_sums(om, u[m], r, Jp, dTp);
                    const cd gl = band_glin(f, ak, r);
                    if (GRAD) {
                        u[m] = gl;
                    } else {
                        const double sm = band_step(f, ak, dtau, scheme);
                        u[m] = cd{__builtin_fma(sm, gl.x, u[m].x), __builtin_fma(sm, gl.y, u[m].y)};  // U1
                        s[m] = sm * invN;
                    }
                    x = cd{-f.q * r.y, f.q * r.x};  // i q r
                }
                v[m] = x;
            });
            Jp *= wj;
            dTp *= wj;
            col_sum2<N>(Jp, dTp, nullptr);
            if (col_on && pc.t == 0) {
                part[2 * j] = Jp;
                part[2 * j + 1] = dTp;
            }
            fft_inv<N, PT>(v, exC, twc, pc);
            store_col(xcol);
        }
        __syncthreads();
        // J, dJ/dT and T' from the partials; no other wavefront reads them before the next pass C
        if (wave == R::NT / 64 - 1)
            finalize_loop(s1, 0, w, sc, GRAD ? MODE_GRAD : MODE_STEP, dtau,
                          J_hist ? J_hist + (size_t)st * jstride : nullptr, Jout, dJdTout);
        if (rows_here) {  // pass D: u r_x
            row_gather_raw<G, R::B_ROW>(X, LD, a, a + R::P, pr.t, v);
            fft_inv<M, PT, true>(v, exD, twr, pr);
#pragma unroll
            for (int m = 0; m < PT; ++m) v[m] = cd{ug[m].x * v[m].x, ug[m].y * v[m].y};
            fft_fwd<M, PT, true>(v, exD, twr, pr);
            res_split<M, N, false, false>(L, v, exD + pr.xs * R::ZS, pr.t, X, a, row_on);
        }
        __syncthreads();
        if (cols_here) load_col();
        if constexpr (R::SPLIT) __syncthreads();  // X has been read: its space may be used
        if (cols_here) {  // pass E, and the next step's pass A
            fft_fwd<N, PT>(v, exE, twc, pc);
#pragma unroll
            for (int m = 0; m < PT; ++m) u[m] = GRAD ? band_g1(u[m], v[m], invN) : band_update(u[m], v[m], s[m]);
            static_for<PT>([&](auto mc) {  // slots outside the band stay zero
                constexpr int m = decltype(mc)::value;
                if (!(col_on && BandSlot<N, m>::in(pc.t))) u[m] = cd{0.0, 0.0};
            });
            if (!GRAD && st + 1 < nsteps) inverse_u();
        }
        __syncthreads();
    }
    // the band values through LDS (over A), then every entry of the rfft layout
    static_for<PT>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        using B = BandSlot<N, m>;
        if (col_on && B::in(pc.t)) A[j * R::NB + B::kk(pc.t)] = u[m];
    });
    __syncthreads();
    for (int i = tid; i < N * R::H; i += R::NT) {
        const int e = i / R::H, jj = i % R::H;
        const int kk = jj < R::C ? band_row(e, N, R::Ks) : -1;
        dst[i] = kk >= 0 ? A[jj * R::NB + kk] : cd{0.0, 0.0};
    }
    if (!GRAD && tid == 0) *T = sc[0];
}

}  // namespace lo
