// LDS-resident form of the fictitious-time step (Sec. 4.2): one block holds one loop's band
// state and its two live intermediates in LDS and runs every pass of every step in one
// launch, so HBM sees only the state's load and store. It applies where a loop's working
// set fits in the 160 KB of LDS of a CU (for example 32 x 256, 64 x 128, 128 x 64).
//
// The column passes are the HBM form's own pass bodies (col_pass_A/C/E) pointed at LDS
// arrays. The row passes are restated here to read and write the resident arrays directly
// instead of staging tiles, with the same row pairing, transforms, products and split, and
// the per-loop sums use the same fixed order. A step therefore gives the same bits as the
// HBM form.
//
// LDS carve (complex values unless noted), for a loop of M x N (Nx x Ns):
//   U  [C][NB]   band state; pass C overwrites it with U1 = u + dtau sigma G_lin, pass E
//                with the new state (each element is read before it is written, by one thread)
//   A  [C][N+1]  u after the inverse s-transforms (pass A, or E fused with the next A)
//   X  [C][N+1]  B, then C (in place, column by column), then D (in place, pair by pair)
//   EX           exchange regions: ColG<N>::LDS for the column passes, or one region of XS values
//                per pair of rows for the row passes
//   2C doubles   per-column partial sums of J and dJ/dT
//   12 doubles   T, T_old, J, dJ/dT and the two-wavefront reduction slots
// Columns of A and X are N + 1 apart: a row pass reads 16 columns of a row, or a short column
// pass a point of 16 columns, at a time, and the odd stride puts them on different banks.
#pragma once

#include "passes.hpp"

namespace lo {

template <int M, int N>
struct ResG {
    static constexpr int C = (M - 1) / 3 + 1;
    static constexpr int Ks = (N - 1) / 3;
    static constexpr int NB = 2 * Ks + 1;
    static constexpr int LD = N + 1;
    static constexpr int W = C * LD;
    static constexpr int S = C * NB;
    // Row pass lanes are mapped pair-fastest (XLOW), so that consecutive lanes touch
    // consecutive rows of A and X.
    static constexpr int RX = RowG<M>::P * Fft<M, RowG<M>::PT, true>::XS;
    static constexpr int EX = ColG<N>::LDS > RX ? ColG<N>::LDS : RX;
    static constexpr int DOUBLES = 2 * C + 12;
    static constexpr size_t BYTES = sizeof(cd) * (size_t)(S + 2 * W + EX) + sizeof(double) * DOUBLES;
    static constexpr bool FITS = BYTES <= 160 * 1024 && N <= 512 && M <= 128;
    // Two blocks share a CU where both fit its LDS; the kernel is then compiled for two
    // wavefronts per SIMD (at most 256 registers each, a few spilled), which costs a lone
    // block 5-8% but lets a second loop hide the first one's latency.
    static constexpr int BLOCKS_PER_CU = BYTES <= 80 * 1024 ? 2 : 1;
    static constexpr int COL_ROUNDS = (C + ColG<N>::F - 1) / ColG<N>::F;
    static constexpr int ROW_ROUNDS = (N + RowG<M>::ROWS - 1) / RowG<M>::ROWS;
};

// F + i G of rows a and b of a resident [j][n] array (zero for rows past the loop, as the HBM
// form stages them) in the slots of a thread.
template <int M>
__device__ __forceinline__ void res_gather(const Shape& sh, const cd* X, int t, int a, int b, bool oka, bool okb,
                                           cd* v) {
    using G = RowG<M>;
    if (okb) {
        row_gather_raw<G, true>(X, sh.ld, a, b, t, v);
    } else {
        row_gather_raw<G, false>(X, sh.ld, oka ? a : 0, 0, t, v);
        if (!oka)
#pragma unroll
            for (int m = 0; m < G::PT; ++m) v[m] = cd{0.0, 0.0};
    }
}

// Split of the products' spectrum (slots va) into rows a and b of X, through the pair's region.
template <int M, bool DX>
__device__ __forceinline__ void res_split(const Shape& sh, const cd* va, cd* ex, const FftPos<M, RowG<M>::PT, true>& pos,
                                          cd* X, int a, int b, bool oka, bool okb) {
    using G = RowG<M>;
    cd* z = ex + pos.xs * Fft<M, G::PT, true>::XS;
    row_put<G>(z, pos.t, va);
    wave_lds_order();
    for (int j = pos.t; j < G::CMAX; j += G::TPF) {
        cd wa, wb;
        row_split<M, DX>(sh.L, j, z[j], z[j == 0 ? 0 : M - G::SH - j], wa, wb);
        if (oka) X[j * sh.ld + a] = wa;
        if (okb) X[j * sh.ld + b] = wb;
    }
    wave_lds_order();  // the exchange region is reused by this group's next transform
}

// Pass B for the pairs of row tile `tile`: X = (u u_x) = (1/2) (u^2)_x per row, from A.
template <int M>
__device__ __forceinline__ void res_row_B(const Shape& sh, int tile, const cd* A, cd* X, cd* exr,
                                          const cd* __restrict__ tw) {
    using G = RowG<M>;
    static_assert(M <= kSquareMaxM, "the resident form takes the square form of u u_x");
    const FftPos<M, G::PT, true> pos(threadIdx.x);
    const int a = tile * G::ROWS + pos.xs, b = a + G::P;
    const bool oka = a < sh.N, okb = b < sh.N;
    TwCache<M, G::PT> twc;
    tw_cache_load<M, G::PT>(twc, pos, tw);
    cd va[G::PT];
    res_gather<M>(sh, A, pos.t, a, b, oka, okb, va);
    row_square<M, G::PT, true>(va, exr, twc, pos);
    wave_lds_order();
    res_split<M, true>(sh, va, exr, pos, X, a, b, oka, okb);
}

// Pass D for the pairs of row tile `tile`: X = (u r_x) per row, from A and X (r_x), in place.
template <int M>
__device__ __forceinline__ void res_row_D(const Shape& sh, int tile, const cd* A, cd* X, cd* exr,
                                          const cd* __restrict__ tw) {
    using G = RowG<M>;
    const FftPos<M, G::PT, true> pos(threadIdx.x);
    const int a = tile * G::ROWS + pos.xs, b = a + G::P;
    const bool oka = a < sh.N, okb = b < sh.N;
    TwCache<M, G::PT> twc;
    tw_cache_load<M, G::PT>(twc, pos, tw);
    cd va[G::PT], vb[G::PT];
    res_gather<M>(sh, A, pos.t, a, b, oka, okb, va);
    res_gather<M>(sh, X, pos.t, a, b, oka, okb, vb);
    // every read of rows a and b of X (by this group only) precedes the group's writes below
    row_product<M, G::PT, true>(va, vb, exr, twc, pos);
    wave_lds_order();
    res_split<M, false>(sh, va, exr, pos, X, a, b, oka, okb);
}

}  // namespace lo
