// Initial loops from chaotic Kuramoto-Sivashinsky runs (Sec. 4.3): the KS equation
// u_t = -u u_x - u_xx - u_xxxx (eq. KS) integrated by ETDRK4 on its Fourier-Galerkin system,
// the norm ||u||(t) (eq. conventinal_L2norm) recorded along the runs, pairs of its maxima
// that nearly repeat, and the temporal low-pass that turns a segment into a loop.
//
// A run's state is a few dozen modes, so the whole state, the ETDRK4 coefficients and the stage
// values stay in registers, NX/8 lanes per run, and the two transforms of each nonlinear
// evaluation run through fft.hpp. HBM sees only the samples.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "fft.hpp"
#include "ks_initial_loops.h"

namespace {

using lo::cd;

constexpr double kTwoPi = 6.283185307179586476925286766559;

// ----------------------------------------------------------------------------- ETDRK4
// phi_1..3 of z (phi_k(z) = sum_n z^n / (n + k)!): the series below |z| = 1, the recurrence
// phi_{k+1} = (phi_k - 1/k!) / z from phi_0 = e^z above (no cancellation worse than a factor
// of a few there).
__device__ void phis(double z, double& p1, double& p2, double& p3) {
    if (fabs(z) < 1.0) {
        // Horner over n = 24 .. 0 of z^n / (n + k)!, with 1/(n + k)! formed downwards
        double f = 1.0;  // 1/27!, built upwards once
        for (int i = 2; i <= 27; ++i) f /= (double)i;
        double inv[28];
        inv[27] = f;
        for (int i = 27; i >= 1; --i) inv[i - 1] = inv[i] * (double)i;
        double a1 = 0.0, a2 = 0.0, a3 = 0.0;
        for (int n = 24; n >= 0; --n) {
            a1 = a1 * z + inv[n + 1];
            a2 = a2 * z + inv[n + 2];
            a3 = a3 * z + inv[n + 3];
        }
        p1 = a1;
        p2 = a2;
        p3 = a3;
    } else {
        p1 = expm1(z) / z;
        p2 = (p1 - 1.0) / z;
        p3 = (p2 - 0.5) / z;
    }
}

struct Etd {
    double E, E2, Q, f1, f2, f3, q;
};

// Coefficients of mode j (Cox & Matthews): z = h c_j, c_j = q^2 - q^4,
// Q = (h/2) phi_1(z/2), f1 = h (phi_1 - 3 phi_2 + 4 phi_3), f2 = h (phi_2 - 2 phi_3),
// f3 = h (4 phi_3 - phi_2).
__device__ Etd etd_coeffs(int j, double L, double h) {
    Etd e;
    e.q = kTwoPi * j / L;
    const double q2 = e.q * e.q;
    const double c = q2 - q2 * q2;
    const double z = h * c;
    double p1, p2, p3, h1, h2, h3;
    phis(z, p1, p2, p3);
    phis(0.5 * z, h1, h2, h3);
    e.E = exp(z);
    e.E2 = exp(0.5 * z);
    e.Q = 0.5 * h * h1;
    e.f1 = h * (p1 - 3.0 * p2 + 4.0 * p3);
    e.f2 = h * (p2 - 2.0 * p3);
    e.f3 = h * (4.0 * p3 - p2);
    return e;
}

// Runs of NX points on TPF = NX/8 lanes each, one wavefront per block. Lane t of a run holds the
// modes e = t + TPF m, m = 0, 1, 2 (NX/3 > K >= e covers no more), zero beyond K.
//
// What bounds a step is the chain of its eight transforms in one wavefront: instruction
// issue (about 930 vector instructions of 4 cycles) and the latency of one LDS exchange per
// transform; even 4096 runs are only two wavefronts per CU. So the transforms leave out what
// is known to vanish: the field is the real part of U_0 + 2 sum_{j>=1} U_j e^{i q x}, so the
// inverse takes five zero slots of eight and only its real part is formed; the forward of
// the real square is needed in the same three slots. Runs do not share a transform (two
// rows as real and imaginary part would): a run that overflows leaves its neighbours alone.
// 4096 runs of 64 modes: 3.1 us per step (3.4 with the twiddle powers formed in every transform); as
// direct sums, one wavefront per run, 18.1.
template <int NX>
struct Dns {
    static constexpr int K = (NX - 1) / 3;
    static constexpr int H = NX / 2 + 1;
    using E = lo::Fft<NX, 8>;
    static constexpr int TPF = E::TPF, RUNS = E::XPW;  // lanes per run, runs per wavefront
    static constexpr int R = 3;                        // modes per lane
    static_assert(3 * TPF > K && TPF <= 64, "the band fits three slots");
};

// Inverse DFT of 8 values whose inputs 3 .. 7 are zero (v[0..2] in, v[0..7] out).
__device__ __forceinline__ void dft8_inv_low3(cd* v) {
    const cd x0 = v[0], x1 = v[1], x2 = v[2], r2 = lo::rot90<true>(x2);
    const cd e0 = lo::cadd(x0, x2), e2 = lo::csub(x0, x2), e1 = lo::cadd(x0, r2), e3 = lo::csub(x0, r2);
    const cd o1 = lo::w16<true, 2>(x1), o2 = lo::rot90<true>(x1), o3 = lo::w16<true, 6>(x1);
    v[0] = lo::cadd(e0, x1);
    v[4] = lo::csub(e0, x1);
    v[1] = lo::cadd(e1, o1);
    v[5] = lo::csub(e1, o1);
    v[2] = lo::cadd(e2, o2);
    v[6] = lo::csub(e2, o2);
    v[3] = lo::cadd(e3, o3);
    v[7] = lo::csub(e3, o3);
}

// Forward DFT of 8 real values (g in, v out).
__device__ __forceinline__ void dft8_fwd_real(const double* g, cd* v) {
    const double a0 = g[0] + g[4], a1 = g[0] - g[4], a2 = g[2] + g[6], a3 = g[2] - g[6];
    const double b0 = g[1] + g[5], b1 = g[1] - g[5], b2 = g[3] + g[7], b3 = g[3] - g[7];
    const double e0 = a0 + a2, e2 = a0 - a2, o0 = b0 + b2, o2 = b0 - b2;
    const double c = (b1 - b3) * lo::kSqrtHalf, d = (b1 + b3) * lo::kSqrtHalf;
    v[0] = cd{e0 + o0, 0.0};
    v[4] = cd{e0 - o0, 0.0};
    v[2] = cd{e2, -o2};
    v[6] = cd{e2, o2};
    v[1] = cd{a1 + c, -a3 - d};
    v[7] = cd{a1 + c, a3 + d};
    v[5] = cd{a1 - c, d - a3};
    v[3] = cd{a1 - c, a3 - d};
}

// N_hat_j = -(i q_j / 2) FFT(u^2)_j for the lane's modes, from its band values v. hs: q_j / (2 NX).
template <int NX>
__device__ __forceinline__ void nonlinear(const cd (&v)[3], const double (&hs)[3], const double two0, cd (&out)[3],
                                          cd* ex, const lo::TwCache<NX, 8, true>& c, const lo::FftPos<NX, 8>& p) {
    using E = lo::Fft<NX, 8>;
    cd w[8];
    w[0] = cd{two0 * v[0].x, two0 * v[0].y};  // 2 U_j, and U_0
    w[1] = cd{2.0 * v[1].x, 2.0 * v[1].y};
    w[2] = cd{2.0 * v[2].x, 2.0 * v[2].y};
    // lo::fft_inv with the zero inputs left out
    dft8_inv_low3(w);
    if constexpr (E::L >= 2) {
        lo::apply_twiddles<8, 1, true, true, lo::FORMED>(w, 0, c.w[1]);
        lo::exchange<NX, 8, false, 1, false>(w, ex, p);
        lo::dft_pt<8, true>(w);
    }
    if constexpr (E::F > 1) {
        lo::apply_twiddles<8, 1, true, true, lo::FORMED>(w, 0, c.w[0]);
        lo::swap_f<8, E::F>(w);
        lo::dft_f<8, E::F, true>(w);
    }
    if constexpr (E::F == 1) {  // lo::fft_fwd of the real squares
        double g[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) g[m] = w[m].x * w[m].x;
        dft8_fwd_real(g, w);
        if constexpr (E::L >= 2) {
            lo::exchange<NX, 8, false, 1, true>(w, ex, p);
            lo::apply_twiddles<8, 1, false, true, lo::FORMED>(w, 0, c.w[1]);
            lo::dft_pt<8, false>(w);
        }
    } else {
#pragma unroll
        for (int m = 0; m < 8; ++m) w[m] = cd{w[m].x * w[m].x, 0.0};
        lo::fft_fwd<NX, 8>(w, ex, c, p);
    }
#pragma unroll
    for (int r = 0; r < 3; ++r) out[r] = cd{hs[r] * w[r].y, -hs[r] * w[r].x};
}

// Stores the modes of a run (zero beyond K) into a row of H values; y0: imaginary part of the mean,
// which u holds apart as zero, or as NaN once the run has overflowed.
template <int NX>
__device__ __forceinline__ void store_modes(const cd (&u)[3], double y0, int t, cd* row) {
    using D = Dns<NX>;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const int j = t + r * D::TPF;
        if (j <= D::K) row[j] = cd{u[r].x, j == 0 ? y0 + u[r].y : u[r].y};
    }
    for (int j = D::K + 1 + t; j < D::H; j += D::TPF) row[j] = cd{0.0, 0.0};
}

// nsteps ETDRK4 steps of the runs of one wavefront.
template <int NX>
__global__ __launch_bounds__(64) void k_ks_etdrk4(double L, int sym, double h, int nsteps, int every, int ntraj,
                                                  cd* uhat, double* norms, cd* snaps, int stride) {
    using D = Dns<NX>;
    __shared__ __align__(16) cd ex[D::RUNS * D::E::XS];
    __shared__ Etd tab[D::K + 1];
    const int lane = threadIdx.x;
    const lo::FftPos<NX, 8> p(lane);
    const int t = p.t;
    const size_t run = (size_t)blockIdx.x * D::RUNS + p.xs;
    const bool live = run < (size_t)ntraj;
    for (int j = lane; j <= D::K; j += 64) tab[j] = etd_coeffs(j, L, h);
    lo::TwCache<NX, 8, true> twc;
#pragma unroll
    for (int i = 0; i < D::E::L; ++i) {
        const int span = i == 0 ? D::E::F : D::E::F * 8;  // as lo::tw_cache_load, at most two stages
        const int ti = i == D::E::L - 1 ? p.t : p.f0;
#pragma unroll
        for (int m : {1, 2, 3, 4, 8}) {
            double sn, cs;
            sincospi(-2.0 * (double)(ti * m) / (double)(span * 8), &sn, &cs);
            twc.w[i][m - 1] = cd{cs, sn};
        }
        if (i == 0)
            lo::tw_powers<D::E::F == 4 ? lo::TURNED_4 : lo::WITH_W3>(twc.w[i]);  // F = 2: w^4 is a quarter turn
        else
            lo::tw_powers<lo::WITH_W3>(twc.w[i]);
    }
    __syncthreads();
    Etd co[3];
    double hs[3];
    cd u[3];
    double y0 = 0.0;
    cd* ur = uhat + (live ? run : 0) * D::H;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const int j = t + r * D::TPF;
        const bool in = live && j <= D::K;
        co[r] = in ? tab[j] : Etd{0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        hs[r] = 0.5 * co[r].q / NX;
        u[r] = in ? ur[j] : cd{0.0, 0.0};
        if (sym) u[r].x = 0.0;
    }
    // the field takes the real part of the mean mode; its imaginary part, which no step changes,
    // is only handed on
    const double two0 = t == 0 ? 1.0 : 2.0;
    if (t == 0) {
        y0 = u[0].y;
        u[0].y = 0.0;
    }
    int left = 0, i_s = 0;  // steps to the next sample, its index
    for (int i = 0; i < nsteps; ++i) {
        if (left == 0) {
            left = every;
            if (norms || snaps) {
                double e = 0.0;
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    const bool mean = r == 0 && t == 0;
                    const double y = mean ? y0 + u[r].y : u[r].y;
                    e += (mean ? 1.0 : 2.0) * (u[r].x * u[r].x + y * y);
                }
                if constexpr (D::E::L == 1) {  // a run's lanes are equal modulo RUNS
                    for (int o = 32; o >= 64 / D::TPF; o >>= 1) e += __shfl_xor(e, o, 64);
                } else {
                    for (int o = D::TPF / 2; o > 0; o >>= 1) e += __shfl_xor(e, o, 64);
                }
                const size_t row = run * (size_t)stride + i_s;
                if (live && norms && t == 0) norms[row] = sqrt(L * e);
                if (live && snaps) store_modes<NX>(u, y0, t, snaps + row * D::H);
            }
            ++i_s;
        }
        --left;
        cd Nu[3], Na[3], Nb[3], Nc[3], a[3], b[3], c[3];
        nonlinear<NX>(u, hs, two0, Nu, ex, twc, p);
#pragma unroll
        for (int r = 0; r < 3; ++r)
            a[r] = cd{co[r].E2 * u[r].x + co[r].Q * Nu[r].x, co[r].E2 * u[r].y + co[r].Q * Nu[r].y};
        nonlinear<NX>(a, hs, two0, Na, ex, twc, p);
#pragma unroll
        for (int r = 0; r < 3; ++r)
            b[r] = cd{co[r].E2 * u[r].x + co[r].Q * Na[r].x, co[r].E2 * u[r].y + co[r].Q * Na[r].y};
        nonlinear<NX>(b, hs, two0, Nb, ex, twc, p);
#pragma unroll
        for (int r = 0; r < 3; ++r)
            c[r] = cd{co[r].E2 * a[r].x + co[r].Q * (2.0 * Nb[r].x - Nu[r].x),
                      co[r].E2 * a[r].y + co[r].Q * (2.0 * Nb[r].y - Nu[r].y)};
        nonlinear<NX>(c, hs, two0, Nc, ex, twc, p);
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const Etd& e = co[r];
            cd n;
            n.x = e.E * u[r].x + e.f1 * Nu[r].x + 2.0 * e.f2 * (Na[r].x + Nb[r].x) + e.f3 * Nc[r].x;
            n.y = e.E * u[r].y + e.f1 * Nu[r].y + 2.0 * e.f2 * (Na[r].y + Nb[r].y) + e.f3 * Nc[r].y;
            if (sym) n.x = 0.0;
            u[r] = n;
        }
    }
    if (live) store_modes<NX>(u, y0, t, ur);
}

// ------------------------------------------------------------------------- recurrences
__device__ __forceinline__ bool is_max(const double* n, int i, int ns) {
    return i >= 1 && i <= ns - 2 && n[i - 1] < n[i] && n[i] >= n[i + 1];
}

// pairs (a, b) of maxima of run blockIdx.x starting at maximum a, in increasing b; with
// out == nullptr only counted. peak(b): whether sample b is a maximum.
template <class Peak>
__device__ int scan_from(const double* n, int a, int ns, double dt_s, double tol, double Tmin, double Tmax,
                         int2* out, int base, int cap, Peak&& peak) {
    int c = 0;
    for (int b = a + 1; b <= ns - 2; ++b) {
        const double T = (double)(b - a) * dt_s;
        if (T > Tmax) break;
        if (T >= Tmin && peak(b) && fabs(n[b] - n[a]) <= tol * n[a]) {
            if (out && base + c < cap) out[base + c] = make_int2(a, b);
            ++c;
        }
    }
    return c;
}

constexpr int kScanBlock = 256;
constexpr int kMaxList = 2048;  // maxima of a run kept in LDS

// Exclusive prefix sum of v over the block (in thread order); total: the block's sum.
__device__ __forceinline__ int block_scan(int v, int* sums, int& total) {
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    int x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) sums[wave] = x;
    __syncthreads();
    int before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < kScanBlock / 64; ++w) {
        if (w < wave) before += sums[w];
        total += sums[w];
    }
    __syncthreads();
    return before + x - v;
}

// One block per run. The run's maxima (one sample in tens) are listed in LDS, in order; a
// wavefront then tests the pairs of one maximum a against 64 later ones at a time, once to
// count them, and once more, after a prefix sum over the maxima, to write them. Walking every
// sample after each maximum instead is a chain of dependent loads: with ks_segments_to_loops on
// 128 runs of 2000 samples and 256 loops it took 3539 us for the two, against 47.
// A run of more than kMaxList maxima takes that walk: tiles of 256 candidate samples a, each
// thread counts its pairs, an exclusive scan over the tile places them. The list's LDS, which leaves
// a CU half the wavefronts that the walk alone could have, then holds a bit per sample that says
// which are maxima, up to 64 kMaxList samples: 4096 runs of 20000 samples of noise take 18100 us,
// 24900 without the bits and 22600 on the full CU.
__global__ __launch_bounds__(kScanBlock) void k_ks_recurrences(const double* norms, int stride, int ns, double dt_s,
                                                               double tol, double Tmin, double Tmax, int cap,
                                                               int2* pairs, int* counts) {
    __shared__ int sums[kScanBlock / 64];
    __shared__ double val[kMaxList];
    __shared__ int idx[kMaxList], cnt[kMaxList];
    const double* n = norms + (size_t)blockIdx.x * stride;
    int2* out = pairs + (size_t)blockIdx.x * cap;
    const int t = threadIdx.x, lane = t % 64, wave = t / 64;
    int nm = 0;  // maxima so far
    for (int a0 = 0; a0 < ns; a0 += kScanBlock) {
        const int a = a0 + t;
        const bool m = a < ns && is_max(n, a, ns);
        int total;
        const int at = nm + block_scan(m, sums, total);
        if (m && at < kMaxList) {
            idx[at] = a;
            val[at] = n[a];
        }
        nm += total;
    }
    __syncthreads();
    if (nm <= kMaxList) {
        // pairs (a, b) of the maximum at position i of the list with later ones, in order of b;
        // write >= 0: stored from pair number write on. Returns their count (all lanes).
        auto scan = [&](int i, int write) {
            const int a = idx[i];
            const double va = val[i];
            int c = 0;
            for (int k0 = i + 1; k0 < nm; k0 += 64) {
                const int k = k0 + lane;
                const double T = k < nm ? (double)(idx[k] - a) * dt_s : 0.0;
                const bool in = k < nm && !(T > Tmax);
                const bool hit = in && T >= Tmin && fabs(val[k] - va) <= tol * va;
                const unsigned long long hits = __ballot(hit);
                if (write >= 0 && hit) {
                    const int at = write + c + __popcll(hits & ((1ull << lane) - 1));
                    if (at < cap) out[at] = make_int2(a, idx[k]);
                }
                c += __popcll(hits);
                if (__ballot(in) != ~0ull) break;  // the rest lies beyond Tmax, or past the list
            }
            return c;
        };
        for (int i = wave; i < nm; i += kScanBlock / 64) {
            const int c = scan(i, -1);
            if (lane == 0) cnt[i] = c;
        }
        __syncthreads();
        int base = 0;
        for (int i0 = 0; i0 < nm; i0 += kScanBlock) {  // counts -> first pair numbers
            const int i = i0 + t;
            int total;
            const int c = i < nm ? cnt[i] : 0;
            const int at = base + block_scan(c, sums, total);
            if (i < nm) cnt[i] = c > 0 ? at : -1;
            base += total;
        }
        __syncthreads();
        for (int i = wave; i < nm; i += kScanBlock / 64)
            if (cnt[i] >= 0 && cnt[i] < cap) scan(i, cnt[i]);
        if (t == 0) counts[blockIdx.x] = base;
        return;
    }
    auto walk = [&](auto&& peak) {
        int base = 0;
        for (int a0 = 0; a0 < ns; a0 += kScanBlock) {
            const int a = a0 + t;
            const bool m = a < ns && peak(a);
            const int c = m ? scan_from(n, a, ns, dt_s, tol, Tmin, Tmax, nullptr, 0, 0, peak) : 0;
            int total;
            const int at = base + block_scan(c, sums, total);
            if (m && c > 0) scan_from(n, a, ns, dt_s, tol, Tmin, Tmax, out, at, cap, peak);
            base += total;
        }
        if (t == 0) counts[blockIdx.x] = base;
    };
    if (ns <= 64 * kMaxList) {
        unsigned long long* bits = reinterpret_cast<unsigned long long*>(val);
        __syncthreads();  // every thread has left the list
        for (int a0 = 0; a0 < ns; a0 += kScanBlock) {
            const unsigned long long m = __ballot(a0 + t < ns && is_max(n, a0 + t, ns));
            if (lane == 0 && a0 + t < ns) bits[(a0 + t) / 64] = m;
        }
        __syncthreads();
        walk([&](int b) { return (bits[b / 64] >> (b % 64) & 1) != 0; });
    } else {
        walk([&](int b) { return is_max(n, b, ns); });
    }
}

// ------------------------------------------------------------------- segments to loops
// One block per loop. c_{j,k} = (1/n) sum_i u_hat_j(t_{a+i}) e^{-2 pi i k i / n} for |k| <= kc,
// j <= Kx (0 elsewhere) from the sums C_jk = sum_i u_hat_j cos and S_jk = sum_i u_hat_j sin of
// 2 pi k i / n, which give both signs of k: c_{j,+-k} = (C -+ i S) / n. Eight lanes share an item,
// (j, four k's), each taking every eighth sample, so a sample is loaded once for four k's
// and the lanes' sums are added in a fixed order. The n roots of unity sit in LDS: evaluating
// sincospi per term, as one thread per (j, k) did, costs two hundred instructions instead of one
// LDS read, and is kept only where the roots do not fit (n > kRoots). With kc = 0 the sums are
// plain ones and need no root: forming the item's three unused modes from sincospi there took 4000
// us for 2000 loops of 64 x 64 cut from segments of 5000 samples, against 628 without (before
// the roots were tabulated 2183).
constexpr int kSegBlock = 1024, kSegLanes = 8, kSegK = 4, kRoots = 4096;

__global__ __launch_bounds__(kSegBlock) void k_ks_segments(const cd* snaps, int H, int ntraj, int ns, int stride,
                                                           const int* triples, double dt_s, int Ns, int kc, cd* loops,
                                                           double* T) {
    __shared__ __align__(16) cd root[kRoots];  // e^{2 pi i m / n}
    const int l = blockIdx.x;
    const int tr = triples[3 * l], a = triples[3 * l + 1], b = triples[3 * l + 2];
    const int n = b - a;
    const bool ok = tr >= 0 && tr < ntraj && a >= 0 && b <= ns && n > 2 * kc;
    const int Kx = (2 * (H - 1) - 1) / 3;
    cd* out = loops + (size_t)l * Ns * H;
    if (threadIdx.x == 0) T[l] = ok ? (double)n * dt_s : 0.0;
    for (int e = threadIdx.x; e < Ns * H; e += kSegBlock) {  // entries outside the low-pass
        const int row = e / H, j = e % H;
        const int k = row <= Ns / 2 ? row : row - Ns;
        if (!ok || j > Kx || k < -kc || k > kc) out[e] = cd{0.0, 0.0};
    }
    if (!ok) return;
    const bool table = n <= kRoots;
    auto root_of = [&](int m) {
        double s, c;
        sincospi(2.0 * (double)m / n, &s, &c);
        return cd{c, s};
    };
    if (table && kc > 0)
        for (int m = threadIdx.x; m < n; m += kSegBlock) root[m] = root_of(m);
    __syncthreads();
    const cd* seg = snaps + ((size_t)tr * stride + a) * H;
    const int lane = threadIdx.x % kSegLanes;
    const int items = (Kx + 1) * ((kc + kSegK) / kSegK);
    for (int it0 = 0; it0 < items; it0 += kSegBlock / kSegLanes) {
        const int it = it0 + threadIdx.x / kSegLanes;
        if (it >= items) continue;  // all lanes of the item
        const int j = it % (Kx + 1), k0 = it / (Kx + 1) * kSegK;
        int m[kSegK], step[kSegK];  // (k i) mod n of the lane's next sample
        cd C[kSegK], S[kSegK];
#pragma unroll
        for (int q = 0; q < kSegK; ++q) {
            m[q] = (int)((long long)(k0 + q) * lane % n);
            step[q] = (int)((long long)(k0 + q) * kSegLanes % n);
            C[q] = S[q] = cd{0.0, 0.0};
        }
        auto term = [&](const cd x, const cd w, int q) {
            C[q] = cd{__builtin_fma(x.x, w.x, C[q].x), __builtin_fma(x.y, w.x, C[q].y)};
            S[q] = cd{__builtin_fma(x.x, w.y, S[q].x), __builtin_fma(x.y, w.y, S[q].y)};
        };
        if (kc == 0) {
            for (int i = lane; i < n; i += kSegLanes) term(seg[(size_t)i * H + j], cd{1.0, 0.0}, 0);
        } else if (table) {
#pragma unroll 2
            for (int i = lane; i < n; i += kSegLanes) {
                const cd x = seg[(size_t)i * H + j];
#pragma unroll
                for (int q = 0; q < kSegK; ++q) {
                    term(x, root[m[q]], q);
                    m[q] += step[q];
                    m[q] -= m[q] >= n ? n : 0;
                }
            }
        } else {
            for (int i = lane; i < n; i += kSegLanes) {
                const cd x = seg[(size_t)i * H + j];
#pragma unroll
                for (int q = 0; q < kSegK; ++q) {
                    term(x, root_of(m[q]), q);
                    m[q] = (int)(((long long)m[q] + step[q]) % n);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < kSegK; ++q) {
#pragma unroll
            for (int o = 1; o < kSegLanes; o <<= 1) {
                C[q].x += __shfl_xor(C[q].x, o, 64);
                C[q].y += __shfl_xor(C[q].y, o, 64);
                S[q].x += __shfl_xor(S[q].x, o, 64);
                S[q].y += __shfl_xor(S[q].y, o, 64);
            }
            const int k = k0 + q;
            if (lane == q && k <= kc) {
                out[(size_t)k * H + j] = cd{(C[q].x + S[q].y) / n, (C[q].y - S[q].x) / n};
                if (k > 0) out[(size_t)(Ns - k) * H + j] = cd{(C[q].x - S[q].y) / n, (C[q].y + S[q].x) / n};
            }
        }
    }
}

bool pow2_size(int n, int lo, int hi) { return n >= lo && n <= hi && (n & (n - 1)) == 0; }

template <int NX>
void launch_runs(double L, int sym, double dt, int nsteps, int every, int ntraj, cd* u, double* norms, cd* snaps,
                 int stride, hipStream_t st) {
    constexpr int R = Dns<NX>::RUNS;
    hipLaunchKernelGGL(k_ks_etdrk4<NX>, dim3((ntraj + R - 1) / R), dim3(64), 0, st, L, sym, dt, nsteps, every, ntraj, u,
                       norms, snaps, stride);
}

int hip_status() { return hipGetLastError() == hipSuccess ? LOOP_OK : LOOP_EHIP; }

}  // namespace

extern "C" {

int ks_integrate(double L, int Nx, int ntraj, int symmetric, double dt, int nsteps, int sample_every, double* uhat,
                 double* norms, double* snaps, int sample_stride, void* stream) {
    if (!(L > 0.0) || !std::isfinite(L) || !(dt > 0.0) || !std::isfinite(dt)) return LOOP_EINVAL;
    if (ntraj < 1 || ntraj > 1 << 20 || nsteps < 0 || sample_every < 1 || nsteps % sample_every) return LOOP_EINVAL;
    if (Nx < 8 || Nx > 1024) return LOOP_EINVAL;
    if (!pow2_size(Nx, 16, 256)) return LOOP_ENOTSUP;
    if (!uhat || reinterpret_cast<uintptr_t>(uhat) % 16) return LOOP_EINVAL;
    const int ns = nsteps / sample_every;
    if ((norms || snaps) && sample_stride < ns) return LOOP_EINVAL;
    if ((norms && reinterpret_cast<uintptr_t>(norms) % 8) || (snaps && reinterpret_cast<uintptr_t>(snaps) % 16))
        return LOOP_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    cd* u = reinterpret_cast<cd*>(uhat);
    cd* sn = reinterpret_cast<cd*>(snaps);
    const int sym = symmetric ? 1 : 0;
    switch (Nx) {
        case 16: launch_runs<16>(L, sym, dt, nsteps, sample_every, ntraj, u, norms, sn, sample_stride, st); break;
        case 32: launch_runs<32>(L, sym, dt, nsteps, sample_every, ntraj, u, norms, sn, sample_stride, st); break;
        case 64: launch_runs<64>(L, sym, dt, nsteps, sample_every, ntraj, u, norms, sn, sample_stride, st); break;
        case 128: launch_runs<128>(L, sym, dt, nsteps, sample_every, ntraj, u, norms, sn, sample_stride, st); break;
        case 256: launch_runs<256>(L, sym, dt, nsteps, sample_every, ntraj, u, norms, sn, sample_stride, st); break;
    }
    return hip_status();
}

int ks_recurrences(int ntraj, int nsamples, const double* norms, int sample_stride, double dt_s, double rel_tol,
                   double Tmin, double Tmax, int cap, int* pairs, int* counts, void* stream) {
    if (ntraj < 1 || ntraj > 1 << 20 || nsamples < 0 || sample_stride < nsamples || cap < 0) return LOOP_EINVAL;
    if (!(dt_s > 0.0) || !std::isfinite(dt_s) || !(rel_tol >= 0.0) || !std::isfinite(rel_tol)) return LOOP_EINVAL;
    if (std::isnan(Tmin) || std::isnan(Tmax)) return LOOP_EINVAL;
    if (!norms || !counts || (cap > 0 && !pairs) || reinterpret_cast<uintptr_t>(norms) % 8 ||
        reinterpret_cast<uintptr_t>(pairs) % 8 || reinterpret_cast<uintptr_t>(counts) % 4)
        return LOOP_EINVAL;
    hipLaunchKernelGGL(k_ks_recurrences, dim3(ntraj), dim3(kScanBlock), 0, (hipStream_t)stream, norms,
                       sample_stride, nsamples, dt_s, rel_tol, Tmin, Tmax, cap, reinterpret_cast<int2*>(pairs), counts);
    return hip_status();
}

int ks_segments_to_loops(int Nx, int ntraj, int nsamples, const double* snaps, int sample_stride, int nloops,
                         const int* triples, double dt_s, int Ns, int kc, double* uhat_loops, double* T_loops,
                         void* stream) {
    if (!pow2_size(Nx, 8, 1024) || !pow2_size(Ns, 8, 1024)) return LOOP_EINVAL;
    if (ntraj < 1 || nsamples < 0 || sample_stride < nsamples || nloops < 1 || nloops > 65535) return LOOP_EINVAL;
    if (kc < 0 || kc > (Ns - 1) / 3 || !(dt_s > 0.0) || !std::isfinite(dt_s)) return LOOP_EINVAL;
    if (!snaps || !triples || !uhat_loops || !T_loops || reinterpret_cast<uintptr_t>(snaps) % 16 ||
        reinterpret_cast<uintptr_t>(triples) % 4 || reinterpret_cast<uintptr_t>(uhat_loops) % 16 ||
        reinterpret_cast<uintptr_t>(T_loops) % 8)
        return LOOP_EINVAL;
    hipLaunchKernelGGL(k_ks_segments, dim3(nloops), dim3(kSegBlock), 0, (hipStream_t)stream,
                       reinterpret_cast<const cd*>(snaps), Nx / 2 + 1, ntraj, nsamples, sample_stride, triples, dt_s,
                       Ns, kc, reinterpret_cast<cd*>(uhat_loops), T_loops);
    return hip_status();
}

}  // extern "C"
