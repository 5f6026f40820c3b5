// Double-precision complex FFT building blocks for gfx950 (CDNA4).
//
// A transform of length N = F PT^L (8 <= N <= 1024, F < PT) runs on PT points per thread,
// N/PT threads per transform: one radix-F stage and L radix-PT stages, with a re-distribution
// between stages. Every butterfly's inputs sit in one thread's registers.
//
// A transform pair is (inverse: spectrum -> points) and (forward: points -> spectrum), each
// the mirror of the other, so the points between them can stay in whatever order the
// last inverse stage leaves them in:
//   spectrum layout: thread t holds e = t + m TPF in slot m (TPF = N/PT), natural order;
//   points layout:   slot m = k + F b of a thread holds n = n0 + TPF b + (N/F) k.
// FftPos gives both for a thread, and which of the block's transforms it works on in each.
//
// Re-distribution between stages. What bounds it is the LDS write port: on MI355X a wavefront's
// ds_write_b128 takes 14 cycles of its CU's LDS and its ds_read_b128 4.4 (a 1024-byte access at
// about 64 and 256 bytes per cycle), so a full exchange of 8 values per lane costs about 147
// CU cycles per wavefront, three quarters of them the writes. The radix-F stage therefore
// re-distributes in registers: v_permlane32_swap and v_permlane16_swap exchange a register bit
// with lane bit 5 or 4 (one instruction per pair of dwords), on the vector units of one SIMD
// instead of the LDS that the CU's four SIMDs share. The radix-PT stages exchange
// through LDS: a 256-point transform has one such exchange (4 x 8 x 8), a 32-point one none.
// Against radix 8, 8, 4 with two LDS exchanges (three at 1024 points), on 64 loops of 256 x 1024:
// pass A 29.3 -> 25.9 us, the forward pass C 46.7 -> 41.8, the reverse pass E 45.0 -> 41.0.
//
// The stages between which transforms stay inside one wavefront need no block barrier
// (the LDS performs a wavefront's operations in issue order). A 1024-point transform of 8 points
// per thread spans two wavefronts; its first exchange crosses them, the second does not.
//
// Sign convention: forward uses exp(-2 pi i), inverse exp(+2 pi i). Neither scales.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace lo {

struct cd {
    double x, y;
};

constexpr int TW_N = 4096;  // twiddle table: tw[t] = exp(-2 pi i t / TW_N)

__device__ __forceinline__ cd cadd(cd a, cd b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ cd csub(cd a, cd b) { return {a.x - b.x, a.y - b.y}; }
// Complex product with two fused multiply-adds (explicit, so every kernel that inlines it
// rounds it the same way).
__device__ __forceinline__ cd cmul(cd a, cd b) {
    return {__builtin_fma(a.x, b.x, -(a.y * b.y)), __builtin_fma(a.x, b.y, a.y * b.x)};
}
__device__ __forceinline__ cd cconj(cd a) { return {a.x, -a.y}; }
__device__ __forceinline__ cd cscale(cd a, double s) { return {a.x * s, a.y * s}; }

// multiply by -i (forward) or +i (inverse)
template <bool INV>
__device__ __forceinline__ cd rot90(cd a) {
    return INV ? cd{-a.y, a.x} : cd{a.y, -a.x};
}

constexpr double kSqrtHalf = 0.70710678118654752440084436210484903928;
constexpr double kCos8 = 0.92387953251128675612818318939678828682;  // cos(pi/8)
constexpr double kSin8 = 0.38268343236508977172845998403039886676;  // sin(pi/8)

// multiply by exp(-+ 2 pi i m / 16) for a compile-time m
template <bool INV, int m>
__device__ __forceinline__ cd w16(cd a) {
    constexpr int mm = m % 16;
    if constexpr (mm == 0) {
        return a;
    } else if constexpr (mm == 4) {
        return rot90<INV>(a);
    } else if constexpr (mm == 8) {
        return cd{-a.x, -a.y};
    } else if constexpr (mm == 12) {
        return rot90<!INV>(a);
    } else if constexpr (mm % 4 == 2) {
        // odd multiples of pi/4: (x, y) (c, sy) with |c| = |sy| = sqrt(1/2), one add and one
        // product per component
        constexpr double c = (mm == 2 || mm == 14) ? kSqrtHalf : -kSqrtHalf;
        constexpr double sy = ((mm == 2 || mm == 6) ? kSqrtHalf : -kSqrtHalf) * (INV ? 1.0 : -1.0);
        if constexpr (c == sy) {
            return cd{(a.x - a.y) * c, (a.x + a.y) * c};
        } else {
            return cd{(a.x + a.y) * c, (a.y - a.x) * c};
        }
    } else {
        // cos and sin of 2 pi mm / 16 from the first-octant constants
        constexpr double c = (mm == 1 || mm == 15) ? kCos8 : (mm == 2 || mm == 14) ? kSqrtHalf
                           : (mm == 3 || mm == 13) ? kSin8 : (mm == 5 || mm == 11) ? -kSin8
                           : (mm == 6 || mm == 10) ? -kSqrtHalf : -kCos8;  // 7, 9
        constexpr double s = (mm == 1 || mm == 7) ? kSin8 : (mm == 2 || mm == 6) ? kSqrtHalf
                           : (mm == 3 || mm == 5) ? kCos8 : (mm == 9 || mm == 15) ? -kSin8
                           : (mm == 10 || mm == 14) ? -kSqrtHalf : -kCos8;  // 11, 13
        // forward: exp(-i theta) = (c, -s); inverse: (c, s)
        constexpr double sy = INV ? s : -s;
        return cd{__builtin_fma(a.x, c, -(a.y * sy)), __builtin_fma(a.x, sy, a.y * c)};
    }
}

template <bool INV>
__device__ __forceinline__ void dft2(cd& a, cd& b) {
    cd t = a;
    a = cadd(t, b);
    b = csub(t, b);
}

template <bool INV>
__device__ __forceinline__ void dft4(cd& x0, cd& x1, cd& x2, cd& x3) {
    cd t0 = cadd(x0, x2), t1 = csub(x0, x2), t2 = cadd(x1, x3), t3 = rot90<INV>(csub(x1, x3));
    x0 = cadd(t0, t2);
    x2 = csub(t0, t2);
    x1 = cadd(t1, t3);
    x3 = csub(t1, t3);
}

template <bool INV>
__device__ __forceinline__ void dft8(cd& x0, cd& x1, cd& x2, cd& x3, cd& x4, cd& x5, cd& x6, cd& x7) {
    // radix-2 split over even and odd inputs, each a length-4 DFT
    dft4<INV>(x0, x2, x4, x6);  // E0..E3
    dft4<INV>(x1, x3, x5, x7);  // O0..O3
    const cd o1 = w16<INV, 2>(x3), o2 = w16<INV, 4>(x5), o3 = w16<INV, 6>(x7);
    const cd e0 = x0, e1 = x2, e2 = x4, e3 = x6, o0 = x1;
    x0 = cadd(e0, o0);
    x4 = csub(e0, o0);
    x1 = cadd(e1, o1);
    x5 = csub(e1, o1);
    x2 = cadd(e2, o2);
    x6 = csub(e2, o2);
    x3 = cadd(e3, o3);
    x7 = csub(e3, o3);
}

// 16-point DFT of v[s0 + r * st], r = 0..15 (natural order in and out), as 4 x 4:
// inputs n = 4 n1 + n2, outputs k = k1 + 4 k2.
template <bool INV, int st>
__device__ __forceinline__ void dft16(cd* v, int s0) {
    cd y[16];
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2) {
        cd a = v[s0 + (0 + n2) * st], b = v[s0 + (4 + n2) * st], c = v[s0 + (8 + n2) * st],
           d = v[s0 + (12 + n2) * st];
        dft4<INV>(a, b, c, d);  // over n1: outputs k1 = 0..3
        y[n2 * 4 + 0] = a;
        y[n2 * 4 + 1] = b;
        y[n2 * 4 + 2] = c;
        y[n2 * 4 + 3] = d;
    }
    // twiddle W16^(n2 k1)
    y[1 * 4 + 1] = w16<INV, 1>(y[1 * 4 + 1]);
    y[1 * 4 + 2] = w16<INV, 2>(y[1 * 4 + 2]);
    y[1 * 4 + 3] = w16<INV, 3>(y[1 * 4 + 3]);
    y[2 * 4 + 1] = w16<INV, 2>(y[2 * 4 + 1]);
    y[2 * 4 + 2] = w16<INV, 4>(y[2 * 4 + 2]);
    y[2 * 4 + 3] = w16<INV, 6>(y[2 * 4 + 3]);
    y[3 * 4 + 1] = w16<INV, 3>(y[3 * 4 + 1]);
    y[3 * 4 + 2] = w16<INV, 6>(y[3 * 4 + 2]);
    y[3 * 4 + 3] = w16<INV, 9>(y[3 * 4 + 3]);
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) {
        cd a = y[0 * 4 + k1], b = y[1 * 4 + k1], c = y[2 * 4 + k1], d = y[3 * 4 + k1];
        dft4<INV>(a, b, c, d);  // over n2: outputs k2 = 0..3
        v[s0 + (k1 + 0) * st] = a;
        v[s0 + (k1 + 4) * st] = b;
        v[s0 + (k1 + 8) * st] = c;
        v[s0 + (k1 + 12) * st] = d;
    }
}

// Exact base-2 logarithm of a power of two.
constexpr int ilog2(int n) { return n <= 1 ? 0 : 1 + ilog2(n / 2); }

// XLOW: neighbouring lanes of a wavefront work on different transforms (lane = x + XPW t)
// instead of on neighbouring values of one. For transforms that read and write arrays whose
// fastest index is the transform (rows of an array held column by column in LDS).
template <int N, int PT, bool XLOW = false>
struct Fft {
    static constexpr int LP = ilog2(PT), LN = ilog2(N);
    static constexpr int L = LN / LP;         // radix-PT stages
    static constexpr int LF = LN % LP;        // log2 of the radix of the remaining stage
    static constexpr int F = 1 << LF;
    static constexpr int TPF = N / PT;        // threads per transform
    static constexpr int XPW = TPF >= 64 ? 1 : 64 / TPF;  // transforms per wavefront
    static constexpr bool TWO_WAVES = TPF == 128;
    static_assert(F <= 4 && L >= 1 && L <= 3 && TPF <= 128, "no plan for this length");
    static_assert(L < 3 || F == 1 || TWO_WAVES, "three exchanged stages: one wavefront or two");
    // Strides of the exchange layouts. A b128 access is served 16 lanes at a time on 64 banks
    // of 4 bytes, so 16 consecutive lanes should fall on 16 different 16-byte slots modulo 16:
    // the strides are chosen for that in both directions of each exchange.
    static constexpr int KS = L == 2 ? TPF + 1 : (TWO_WAVES ? 64 : TPF) + 16 / PT;
    static constexpr int K1 = TWO_WAVES ? 2 * PT + 1 : PT + 1;  // first exchange of three stages
    static constexpr int X1 = PT * PT * K1, X2 = (TWO_WAVES ? 2 : 1) * PT * KS;
    // complex values of exchange space per transform (at least N, for other uses of the region)
    static constexpr int XS = L == 1 ? N + 1 : L == 2 ? PT * KS + (XLOW ? 16 / XPW : 0) : (X1 > X2 ? X1 : X2);
};

// Where a thread of a block stands. xs, t: transform and position in the spectrum layout;
// xt, n0: transform and first point in the points layout.
template <int N, int PT, bool XLOW = false>
struct FftPos {
    using E = Fft<N, PT, XLOW>;
    int xs, t, xt, n0;
    int k0, k1, f0, f1;  // digits of the exchanges (f1: with f0, for two wavefronts)
    __device__ __forceinline__ explicit FftPos(int tid) {
        const int lane = tid % 64, wave = tid / 64;
        k0 = k1 = f0 = f1 = 0;
        if constexpr (E::L == 1) {
            f0 = lane / (64 / E::F);
            xs = xt = wave * (64 / E::F) + lane % (64 / E::F);
            t = n0 = f0;
        } else if constexpr (E::TWO_WAVES) {
            // points: lane bits k0 (3), low bits of k1 (2), f0; wavefront: top bit of k1.
            // spectrum: lane bits f0, low bits of f1 (2), f2 (3); wavefront: top bit of f1.
            const int w = wave & 1;
            xs = xt = wave >> 1;
            k0 = lane & 7;
            k1 = ((lane >> 3) & 3) + 4 * w;
            f0 = lane >> 5;
            n0 = k0 + 8 * k1 + 64 * f0;
            f1 = (lane >> 3) + 8 * w;  // between the exchanges: lane bits k0 (3), f0, f1 (2)
            t = (lane & 7) + 8 * w + 16 * (lane >> 3);
        } else if constexpr (E::L == 2) {
            constexpr int X = E::XPW;
            const int in = XLOW ? lane / X : lane;  // lane without the low transform bits
            k0 = in % PT;
            const int rest = in / PT;
            f0 = XLOW ? rest : rest / X;
            xt = wave * X + (XLOW ? lane % X : rest % X);
            n0 = k0 + PT * f0;
            xs = wave * X + (XLOW ? lane % X : lane / E::TPF);
            t = XLOW ? in : lane % E::TPF;
        } else {
            static_assert(E::F == 1 && !XLOW, "");
            xs = xt = tid / E::TPF;
            t = n0 = tid % E::TPF;
            k0 = t % PT;
            k1 = f1 = t / PT;
        }
    }
    // point held in slot m
    __device__ __forceinline__ int point(int m) const {
        return n0 + E::TPF * (m / E::F) + (N / E::F) * (m % E::F);
    }
};

// Per-thread twiddle cache. Stage i (1 .. L, after the radix-F stage) multiplies its input m by
// w^m with w = exp(-2 pi i t_i / (F PT^i)), t_i the position in the spectrum of the stages
// before it. These depend only on the thread, so it loads them once and reuses them for
// every transform it runs. The cache holds w, w^2, w^4 (and w^8) as read from the table, and
// the other powers are formed by one or two complex products, each within a few units in the
// last place. The inverse transform uses the conjugates, after its butterflies, so an error in a
// power's magnitude does not cancel between the two. The stage after the radix-F stage has few
// positions to average such errors over (F of them), and transforms of F > 1 multiply by formed
// powers in one stage more than radix 8 first and F last would. That stage therefore forms its powers
// by quarter turns of the table's, without rounding, where the registers cost no wavefront: with F = 2
// w^4 is such a turn, and w^3 = w^4 conj(w); in 32-point transforms w^8 is one, and w^5, w^6, w^7 =
// w^8 conj(w^3, w^2, w), w^3 from the table. With F = 4 of 256 points, and 16 points per thread, w^3
// alone comes from the table. The cost J of loops whose products outweigh their linear part (rms
// relative error against long double, in units of 1e-16, with all of that stage's powers formed by
// products and now): 16 x 32 4.9 and 2.5, 32 x 32 4.9 and 2.3, 128 x 64 6.5 and 5.7, 256 x 32 6.9 and
// 4.9, at the same speed.
//
// With ALL it holds every power instead, formed once by the same products (equal bit for bit): 16
// registers more per stage, and four products (16 instructions of about 100) less per stage
// of every transform.
enum Powers { FORMED, WITH_W3, TURNED_2, TURNED_4 };  // WITH_W3: FORMED, but w^3 from the table
template <int N, int PT>
constexpr Powers tw_how(int stage) {
    using E = Fft<N, PT>;
    if (PT == 16) return WITH_W3;
    if (PT != 8 || stage != 1 || E::F == 1) return FORMED;
    return E::F == 2 ? TURNED_2 : E::L == 1 ? TURNED_4 : WITH_W3;
}
// Entry b of a stage's cache holds this power: 1, 2, 4 (and 8), then w^3, then w^8.
constexpr int tw_entries(int PT, Powers how) { return ilog2(PT) + (how == WITH_W3 ? 1 : how == TURNED_4 ? 2 : 0); }
constexpr int tw_power(int b, int PT) { return b == ilog2(PT) ? 3 : b > ilog2(PT) ? 8 : 1 << b; }

template <int N, int PT, bool ALL_ = false>
struct TwCache {
    static_assert(!ALL_ || PT == 8, "tw_powers");
    static constexpr bool ALL = ALL_;
    static constexpr int NB = ALL ? PT : ilog2(PT) + 2;
    static constexpr int L = Fft<N, PT>::L;
    cd w[L][NB];
};

// An opaque copy of a cached twiddle: products formed from it are not merged with products
// formed for another transform, so the derived powers do not stay live between transforms.
__device__ __forceinline__ cd opaque(cd w) {
    asm volatile("" : "+v"(w.x), "+v"(w.y));
    return w;
}

template <bool INV>
__device__ __forceinline__ cd cmul_tw(cd a, cd w) {
    return INV ? cd{__builtin_fma(a.x, w.x, a.y * w.y), __builtin_fma(a.y, w.x, -(a.x * w.y))} : cmul(a, w);
}

// w^3, w^5, w^6, w^7 from w, w^2, w^4 (w[m - 1] = w^m), and w^3 and w^8 with some, formed as apply_twiddles forms them
template <Powers HOW>
__device__ __forceinline__ void tw_powers(cd* w) {
    if constexpr (HOW == FORMED) w[2] = cmul(w[0], w[1]);
    if constexpr (HOW == TURNED_2) w[2] = cmul_tw<true>(w[3], w[0]);
    w[4] = HOW == TURNED_4 ? cmul_tw<true>(w[7], w[2]) : cmul(w[0], w[3]);
    w[5] = HOW == TURNED_4 ? cmul_tw<true>(w[7], w[1]) : cmul(w[1], w[3]);
    w[6] = HOW == TURNED_4 ? cmul_tw<true>(w[7], w[0]) : cmul(w[2], w[3]);
#pragma unroll
    for (int b = 0; b < 7; ++b) w[b] = opaque(w[b]);
}

// Table entries of stage i, whose input spectrum positions run over [0, F PT^(i-1)).
template <int N, int PT, int I, bool ALL, class Pos>
__device__ __forceinline__ void tw_cache_fill(TwCache<N, PT, ALL>& c, const Pos& p, const cd* __restrict__ tw) {
    using E = Fft<N, PT>;
    constexpr int span = I == 1 ? E::F : I == 2 ? E::F * PT : E::F * PT * PT;
    if constexpr (span > 1) {
        constexpr int step = TW_N / (span * PT);
        int ti;
        if constexpr (I == E::L) {
            ti = p.t;
        } else if constexpr (I == 1) {
            ti = p.f0;
        } else {
            ti = p.f1;  // the middle stage of three
        }
#pragma unroll
        for (int b = 0; b < tw_entries(PT, tw_how<N, PT>(I)); ++b)
            c.w[I - 1][ALL ? tw_power(b, PT) - 1 : b] = tw[(ti * tw_power(b, PT) * step) & (TW_N - 1)];
        if constexpr (ALL) tw_powers<tw_how<N, PT>(I)>(c.w[I - 1]);
    }
    if constexpr (I < E::L) tw_cache_fill<N, PT, I + 1, ALL>(c, p, tw);
}

template <int N, int PT, bool ALL, class Pos>
__device__ __forceinline__ void tw_cache_load(TwCache<N, PT, ALL>& c, const Pos& p, const cd* __restrict__ tw) {
    tw_cache_fill<N, PT, 1, ALL>(c, p, tw);
}

// Apply w^(k r) to element r of butterfly i (elements in slots i + r NB), from the cache.
template <int R, int NB, bool INV, bool ALL, Powers HOW>
__device__ __forceinline__ void apply_twiddles(cd* v, int i, const cd* base) {
    if constexpr (ALL) {
#pragma unroll
        for (int m = 1; m < R; ++m) v[i + m * NB] = cmul_tw<INV>(v[i + m * NB], base[m - 1]);
        return;
    }
    constexpr int LR = ilog2(R);
    const cd w1 = opaque(base[0]);
    v[i + NB] = cmul_tw<INV>(v[i + NB], w1);
    if constexpr (R >= 4) {
        const cd w2 = opaque(base[1]);
        const cd w3 = HOW == WITH_W3 || HOW == TURNED_4 ? opaque(base[LR])
                      : HOW == TURNED_2                 ? cmul_tw<true>(opaque(base[2]), w1)
                                                        : cmul(w1, w2);
        v[i + 2 * NB] = cmul_tw<INV>(v[i + 2 * NB], w2);
        v[i + 3 * NB] = cmul_tw<INV>(v[i + 3 * NB], w3);
        if constexpr (R >= 8) {
            const cd w4 = opaque(base[2]);
            v[i + 4 * NB] = cmul_tw<INV>(v[i + 4 * NB], w4);
            if constexpr (HOW == TURNED_4) {
                const cd w8 = opaque(base[LR + 1]);
                v[i + 5 * NB] = cmul_tw<INV>(v[i + 5 * NB], cmul_tw<true>(w8, w3));
                v[i + 6 * NB] = cmul_tw<INV>(v[i + 6 * NB], cmul_tw<true>(w8, w2));
                v[i + 7 * NB] = cmul_tw<INV>(v[i + 7 * NB], cmul_tw<true>(w8, w1));
            } else {
                v[i + 5 * NB] = cmul_tw<INV>(v[i + 5 * NB], cmul(w1, w4));
                v[i + 6 * NB] = cmul_tw<INV>(v[i + 6 * NB], cmul(w2, w4));
                v[i + 7 * NB] = cmul_tw<INV>(v[i + 7 * NB], cmul(w3, w4));
            }
            if constexpr (R >= 16) {
                const cd w8 = opaque(base[3]);
                v[i + 8 * NB] = cmul_tw<INV>(v[i + 8 * NB], w8);
#pragma unroll
                for (int m = 1; m < 8; ++m) {
                    const cd wm = (m == 1) ? w1 : (m == 2) ? w2 : (m == 3) ? w3 : (m == 4) ? w4
                                : (m == 5) ? cmul(w1, w4) : (m == 6) ? cmul(w2, w4) : cmul(w3, w4);
                    v[i + (8 + m) * NB] = cmul_tw<INV>(v[i + (8 + m) * NB], cmul(w8, wm));
                }
            }
        }
    }
}

// Wavefront-level LDS ordering. The LDS performs the operations of one wavefront in the order
// they were issued, so a read issued after a write of the same wavefront returns what the
// write stored, for every lane, without waiting for the write to complete (a wait is needed
// only between wavefronts). Only the compiler has to keep the order: no memory operation
// moves across this point. Read results are waited for where they are used.
__device__ __forceinline__ void wave_lds_order() { asm volatile("" ::: "memory"); }

// Ordering between the threads of one transform: wavefront order when it fits in one
// wavefront, otherwise a block barrier (every thread of the block then runs the same code).
template <int TPF>
__device__ __forceinline__ void xsync() {
    if constexpr (TPF <= 64) {
        wave_lds_order();
    } else {
        __syncthreads();
    }
}

template <int PT, bool INV>
__device__ __forceinline__ void dft_pt(cd* v) {
    if constexpr (PT == 16) {
        dft16<INV, 1>(v, 0);
    } else if constexpr (PT == 8) {
        dft8<INV>(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]);
    } else {
        dft4<INV>(v[0], v[1], v[2], v[3]);
    }
}

// Radix-F butterflies over the low bits of the slot index.
template <int PT, int F, bool INV>
__device__ __forceinline__ void dft_f(cd* v) {
#pragma unroll
    for (int b = 0; b < PT; b += F) {
        if constexpr (F == 4) dft4<INV>(v[b], v[b + 1], v[b + 2], v[b + 3]);
        if constexpr (F == 2) dft2<INV>(v[b], v[b + 1]);
    }
}

// Exchange of a register bit with lane bit 5 (W = 32) or 4 (W = 16): lanes whose bit is clear
// keep a and receive their partner's a in b; the others keep b and receive their partner's b
// in a.
template <int W>
__device__ __forceinline__ void swap_dword(unsigned& a, unsigned& b) {
    auto r = W == 32 ? __builtin_amdgcn_permlane32_swap(a, b, false, false)
                     : __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
template <int W>
__device__ __forceinline__ void swap_lane_bit(cd& a, cd& b) {
    unsigned u[4], v[4];
    __builtin_memcpy(u, &a, sizeof(cd));
    __builtin_memcpy(v, &b, sizeof(cd));
#pragma unroll
    for (int i = 0; i < 4; ++i) swap_dword<W>(u[i], v[i]);
    __builtin_memcpy(&a, u, sizeof(cd));
    __builtin_memcpy(&b, v, sizeof(cd));
}
// x + (x of lane ^ O), O a power of two up to 32, without the LDS unit: swaps across rows of 16
// lanes, DPP moves within them. Every lane of the wavefront must be active.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x) {
    unsigned u[2];
    __builtin_memcpy(u, &x, sizeof(x));
#pragma unroll
    for (int i = 0; i < 2; ++i) u[i] = __builtin_amdgcn_update_dpp(0u, u[i], CTRL, 0xf, 0xf, true);
    __builtin_memcpy(&x, u, sizeof(x));
    return x;
}
template <int O>
__device__ __forceinline__ double add_lane_xor(double x) {
    if constexpr (O >= 16) {
        unsigned a[2], b[2];
        __builtin_memcpy(a, &x, sizeof(x));
        __builtin_memcpy(b, &x, sizeof(x));
#pragma unroll
        for (int i = 0; i < 2; ++i) swap_dword<O>(a[i], b[i]);
        double p, q;  // the lane's value and its partner's, in the order of the lane bit
        __builtin_memcpy(&p, a, sizeof(p));
        __builtin_memcpy(&q, b, sizeof(q));
        return p + q;
    } else if constexpr (O == 8) {
        return x + dpp_move<0x128>(x);  // row_ror:8
    } else if constexpr (O == 4) {
        return x + dpp_move<0x1B>(dpp_move<0x141>(x));  // row_half_mirror (xor 7), quad_perm (xor 3)
    } else if constexpr (O == 2) {
        return x + dpp_move<0x4E>(x);  // quad_perm [2, 3, 0, 1]
    } else {
        return x + dpp_move<0xB1>(x);  // quad_perm [1, 0, 3, 2]
    }
}
// Sum over the lanes that agree in all lane bits but FROM, FROM/2 .. TO (xor tree, FROM first).
template <int FROM, int TO = 1>
__device__ __forceinline__ double sum_lanes(double x) {
    if constexpr (FROM >= TO) return sum_lanes<FROM / 2, TO>(add_lane_xor<FROM>(x));
    return x;
}

// Calls f(std::integral_constant<int, m>) for m = 0 .. N-1, unrolled.
template <int N, int M = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (M < N) {
        f(std::integral_constant<int, M>{});
        static_for<N, M + 1>(static_cast<F&&>(f));
    }
}

// The low bits of the slot index (F values) against the top lane bits; its own inverse.
template <int PT, int F>
__device__ __forceinline__ void swap_f(cd* v) {
#pragma unroll
    for (int b = 0; b < PT; b += F) {
        if constexpr (F == 4) {
            swap_lane_bit<16>(v[b], v[b + 1]);
            swap_lane_bit<16>(v[b + 2], v[b + 3]);
            swap_lane_bit<32>(v[b], v[b + 2]);
            swap_lane_bit<32>(v[b + 1], v[b + 3]);
        }
        if constexpr (F == 2) swap_lane_bit<32>(v[b], v[b + 1]);
    }
}

// Exchange S (1 .. L-1) between radix-PT stages S and S + 1 through ex, the exchange space of
// the block's transforms (XS values each). Forward: slot = digit f_S in, digit k_(L-1-S) out.
template <int N, int PT, bool XLOW, int S, bool FWD, class Pos>
__device__ __forceinline__ void exchange(cd* v, cd* ex, const Pos& p) {
    using E = Fft<N, PT, XLOW>;
    // slot of (points-side thread, its register m) and of (spectrum-side thread, its register m)
    auto near_pts = [&](int m) {
        if constexpr (E::L == 2) return p.xt * E::XS + p.k0 * E::KS + p.f0 + E::F * m;
        if constexpr (E::TWO_WAVES && S == 1) return p.xt * E::XS + p.k0 + 8 * (p.k1 * E::K1 + p.f0 + 2 * m);
        if constexpr (E::TWO_WAVES && S == 2) {
            const int w = p.f1 >> 3;
            return p.xt * E::XS + (w * PT + p.k0) * E::KS + (p.f1 & 7) + 8 * m;
        }
        if constexpr (S == 1) return p.xt * E::XS + p.k0 + PT * (p.k1 * E::K1 + m);
        return p.xt * E::XS + p.k0 * E::KS + p.f1 + PT * m;
    };
    auto near_spec = [&](int m) {
        if constexpr (E::L == 2) return p.xs * E::XS + m * E::KS + p.t;
        if constexpr (E::TWO_WAVES && S == 1) {
            return p.xt * E::XS + p.k0 + 8 * (m * E::K1 + p.f1);
        }
        if constexpr (E::TWO_WAVES && S == 2) {
            const int w = p.f1 >> 3;
            return p.xt * E::XS + (w * PT + m) * E::KS + p.k0 + 8 * (p.f1 & 7);
        }
        if constexpr (S == 1) return p.xt * E::XS + p.k0 + PT * (m * E::K1 + p.f1);
        return p.xs * E::XS + m * E::KS + p.t;
    };
    constexpr bool CROSS = E::TWO_WAVES && S == 1;  // the two wavefronts of a transform exchange
    if constexpr (CROSS) __syncthreads();           // the other wavefront may still read its part
#pragma unroll
    for (int m = 0; m < PT; ++m) ex[FWD ? near_pts(m) : near_spec(m)] = v[m];
    if constexpr (CROSS) __syncthreads();
    else wave_lds_order();
#pragma unroll
    for (int m = 0; m < PT; ++m) v[m] = ex[FWD ? near_spec(m) : near_pts(m)];
    if constexpr (CROSS) __syncthreads();
    else wave_lds_order();
}

// Forward transform, points layout in, spectrum layout out. All threads of a wavefront (of
// the block, for transforms of two wavefronts) must call; ex: the block's exchange space.
template <int N, int PT, bool XLOW = false, bool ALL>
__device__ __forceinline__ void fft_fwd(cd* v, cd* ex, const TwCache<N, PT, ALL>& c, const FftPos<N, PT, XLOW>& p) {
    using E = Fft<N, PT, XLOW>;
    if constexpr (E::F > 1) {
        dft_f<PT, E::F, false>(v);
        swap_f<PT, E::F>(v);
        apply_twiddles<PT, 1, false, ALL, tw_how<N, PT>(1)>(v, 0, c.w[0]);
    }
    dft_pt<PT, false>(v);
    if constexpr (E::L >= 2) {
        exchange<N, PT, XLOW, 1, true>(v, ex, p);
        apply_twiddles<PT, 1, false, ALL, tw_how<N, PT>(2)>(v, 0, c.w[1]);
        dft_pt<PT, false>(v);
    }
    if constexpr (E::L >= 3) {
        exchange<N, PT, XLOW, 2, true>(v, ex, p);
        apply_twiddles<PT, 1, false, ALL, tw_how<N, PT>(3)>(v, 0, c.w[2]);
        dft_pt<PT, false>(v);
    }
}

// Inverse transform, spectrum layout in, points layout out.
template <int N, int PT, bool XLOW = false, bool ALL>
__device__ __forceinline__ void fft_inv(cd* v, cd* ex, const TwCache<N, PT, ALL>& c, const FftPos<N, PT, XLOW>& p) {
    using E = Fft<N, PT, XLOW>;
    dft_pt<PT, true>(v);
    if constexpr (E::L >= 3) {
        apply_twiddles<PT, 1, true, ALL, tw_how<N, PT>(3)>(v, 0, c.w[2]);
        exchange<N, PT, XLOW, 2, false>(v, ex, p);
        dft_pt<PT, true>(v);
    }
    if constexpr (E::L >= 2) {
        apply_twiddles<PT, 1, true, ALL, tw_how<N, PT>(2)>(v, 0, c.w[1]);
        exchange<N, PT, XLOW, 1, false>(v, ex, p);
        dft_pt<PT, true>(v);
    }
    if constexpr (E::F > 1) {
        apply_twiddles<PT, 1, true, ALL, tw_how<N, PT>(1)>(v, 0, c.w[0]);
        swap_f<PT, E::F>(v);
        dft_f<PT, E::F, true>(v);
    }
}

}  // namespace lo
