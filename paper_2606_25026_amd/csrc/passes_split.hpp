// The four-pass form of the kick-drift-kick step.  The y axis is factored
// ny = R1 R2 and its transform divided between the z and the x passes, so that
// no pass of its own runs along y:
//
//   z pass   a work-group owns all z of the R1 rows y = y0 + R2 j (fixed x, y0)
//            and transforms z, then j -> k1 (radix R1, twiddle W_ny^(y0 k1));
//            row y0 + R2 k1 of the grid then holds (y0, k1)
//   x pass   a work-group owns all x and the R2 rows y0 (contiguous, fixed k1)
//            of a few z and transforms y0 -> k2 (radix R2, ky = k1 + R1 k2) and
//            x, multiplies, and transforms back to (x, y0)
//   z pass   k1 -> j and z back to real space
//
// Per cell the step then moves 24 (P1) + 16 (kinetic plane pass) + 24 (P5) + 8
// (Green's plane pass) = 72 bytes in four launches instead of 120 in eight:
// the y passes were streams at 6 TB/s with their vector units a third busy, and
// the butterflies they carried fit beside the other passes' traffic.  Step times
// without particles, eight against four passes: 16^3 28.7 / 18.7 us, 64^3 40.7 /
// 29, 128^3 86.5 / 58.4, 192^3 188 / 162, 256^3 328 / 246, 256^3 complex128
// 689 / 546.  Between the passes psi
// and the half spectrum are held in the (y0, k1) form; in real space and
// between calls psi is as ever, the half spectrum stays in the (y0, k1) form.
//
// The half spectrum's kz = 0 and kz = nz/2 planes A and B are real in x and y,
// so rows k1 and R1 - k1 of each say the same, and the two share column 0:
// rows 0 < k1 < R1/2 hold A, rows k1 > R1/2 hold B, and rows 0 and R1/2 (their
// own mirrors) A + iB, which the Green's pass separates by the mode at -k of
// the same tile.  A Nyquist plane of its own took the Green's pass a second
// round of work-groups for 4 tiles of 516 (59 us at 256^3).
#pragma once
#include "passes_common.hpp"

namespace wdm {

// R1 of an axis length (rows of a z-pass group); 0 where the four-pass form is
// not built.  R2 = 4 (16, 32), 8 (64, 96, 128) or 16 (192, 256).
constexpr int y_radix(int n) {
    return n == 16 ? 4 : n == 32 || n == 64 ? 8 : n == 96 || n == 192 ? 12 : n == 128 || n == 256 ? 16 : 0;
}

// x plans of the plane pass by (nx, R2).  A lane holds E values: E / R2 whole y
// columns, or E elements of one x pencil, so R2 divides E; two levels at most,
// one exchange.
template <int N, int R2>
struct XPlanFor {
    using type = typename PlanFor<N>::type;
};
template <> struct XPlanFor<16, 8> { using type = FftPlan<16, 2, 8, 2>; };
template <> struct XPlanFor<16, 16> { using type = FftPlan<16, 1, 16>; };
template <> struct XPlanFor<32, 16> { using type = FftPlan<32, 2, 16, 2>; };
template <> struct XPlanFor<64, 16> { using type = FftPlan<64, 4, 16, 4>; };
template <> struct XPlanFor<96, 4> { using type = FftPlan<96, 4, 12, 8>; };
template <> struct XPlanFor<96, 8> { using type = FftPlan<96, 4, 12, 8>; };
template <> struct XPlanFor<96, 16> { using type = FftPlan<96, 2, 16, 6>; };
template <> struct XPlanFor<192, 4> { using type = FftPlan<192, 8, 24, 8>; };
template <> struct XPlanFor<192, 8> { using type = FftPlan<192, 8, 24, 8>; };
template <> struct XPlanFor<192, 16> { using type = FftPlan<192, 4, 16, 12>; };

// Tile of the plane pass: all x, R2 rows, ZC values of z.  64 pencils (32 at
// nz = 16), so that the 64 lanes of a wavefront take neighbouring pencils and
// one lane index t: the x transform's twiddles and factors are then uniform
// over the wavefront and come through scalar loads instead of the LDS.
template <int NX, int R2, int ZC_, typename T>
struct PlaneTile {
    using FP = typename XPlanFor<NX, R2>::type;
    static_assert(FP::valid() && FP::E % R2 == 0, "x plan");
    static constexpr int ZC = ZC_;
    static constexpr int pencils = R2 * ZC;
    static constexpr int CB = FP::E / R2;
    static constexpr int threads = pencils * FP::T;
    static constexpr int LD = pencils + ZC;           // LDS row of one x
    static constexpr bool uniform = pencils % 64 == 0;
    // Wavefronts per SIMD asked of the compiler: a 1024-lane work-group leaves it
    // room for 128 registers, which it fills by hoisting loads; two of them per
    // CU measured 72 against 97 us for the kinetic pass at 256^3.
    static constexpr int waves = sizeof(T) == 4 && threads == 1024 ? 8 : 1;
};
// Pairs (nx, R2) that have a plane pass.
constexpr bool plane_supported(int nx, int r2) {
    return (nx == 16 || nx == 32 || nx == 64 || nx == 96 || nx == 128 || nx == 192 || nx == 256) &&
           (r2 == 4 || r2 == 8 || r2 == 16);
}
// Values of z in a tile.
constexpr int plane_zc(int r2, int nz) { return r2 == 16 ? 4 : r2 == 8 ? 8 : nz >= 32 ? 16 : 8; }
// Whether the four passes are the faster form for a class with `tiles` plane tiles
// (of all its members) and up to `np` moving particles a member.  A tile lasts 15-30
// us however few there are, the three passes it replaces about 6 us each on a small
// grid.  Step times, eight against four passes, in complex64 without particles:
// nx = 256, 64 tiles 63.2 / 63.5 us (256x64x64), 32 tiles 49.1 / 57.3, 96 tiles 87.4 /
// 77.9; nx = 192, 16 tiles 45.6 / 46.7, 64 tiles 63.3 / 59.4; the 48 values a lane of
// nx = 96 and 192 at R2 = 16, 256 tiles 100.5 / 113.7 (192x256x64), 288 tiles 100.9 / 90.6
// (96x192x96); nx = 128, 16 tiles 41.4 / 36.5; smaller nx are faster at any size
// (32x16x32: 37.7 / 25.3).
// In complex128 few tiles hide less, above all beside many particles: nx = 192, 64
// tiles (192x64x64) 76.1 / 74.6, with 10^5 particles 84 / 92, with 10^6 107 / 113, but with
// 10^4 98 / 94 (192x32x128); nx = 128, 8 tiles (128x16x32) 39.1 / 40.4, with 10^4 57 / 61,
// with 10^6 77 / 81, though with 10^5 65 / 61; 16 tiles (128x32x32) 42.4 / 42.7, with 10^5 67 /
// 63.
// Where those 48 values meet z groups of R1 = 12 rows (ny = 192) the four passes need
// more, the more so the shorter the rows (at nz = 128 a group's columns also leave a
// third of its lanes idle).  complex64, 192x192x128: 128.6 / 137.4 with 384 tiles, 213.8
// / 190.9 with 768.  complex128, one, two and three members: 192x192x96 176.5 / 183.8,
// 294 / 317, 420 / 426 (with 10^6 particles each 216 / 228, 391 / 420, 581 / 602), 192x192x128
// 214 / 228, 378 / 400, 565 / 619, but 192^3 307.5 / 307.2, 588 / 578, 913 / 841; 96x192x128
// 138 / 137, 211 / 211, 290 / 318 (with 10^5 159 / 155, 240 / 228, 336 / 349), but 96x192x96
// 123.7 / 108.8 and 96x192x192 181 / 170.
constexpr bool plane_pays(int nx, int r1, int r2, int nz, int64_t tiles, bool c128, int64_t np) {
    if (r2 == 16 && (nx == 96 || nx == 192)) {
        if (r1 == 12 && nx == 192 && nz <= 128 && (c128 || nz == 128)) return !c128 && tiles >= 768;
        if (r1 == 12 && nx == 96 && nz == 128 && c128) return tiles >= 288 && tiles <= 768;
        return tiles >= 288;
    }
    if (nx == 256) return tiles >= 96;
    if (nx == 192) return tiles >= (c128 && np >= 50000 ? 96 : 64);
    return !(c128 && nx == 128 && nz >= 32 && tiles < 16);
}
// Pairs (nz, R1) that have z passes.
constexpr bool zrows_supported(int nz, int r1) {
    if (y_radix(nz) == 0) return false;   // 384, 512
    if (r1 == 4) return nz <= 64;
    if (r1 == 8) return true;
    return (r1 == 12 || r1 == 16) && nz >= 32;
}

// Column 0 of a group: from the transforms U of a + ib over the group's rows
// (a, b real) to the stored rows, and back.
template <int R1, typename T>
__device__ __forceinline__ void pack_column0(cplx<T>* u) {
#pragma unroll
    for (int k = 1; k < R1 / 2; ++k) {
        const cplx<T> p = u[k], q = u[R1 - k];
        u[k] = cplx<T>{T(0.5) * (p.re + q.re), T(0.5) * (p.im - q.im)};           // A[k]
        u[R1 - k] = cplx<T>{T(0.5) * (q.im + p.im), T(0.5) * (p.re - q.re)};      // B[R1 - k]
    }
}
template <int R1, typename T>
__device__ __forceinline__ void unpack_column0(cplx<T>* u) {
#pragma unroll
    for (int k = 1; k < R1 / 2; ++k) {
        const cplx<T> a = u[k], b = u[R1 - k];
        u[k] = cplx<T>{a.re + b.im, a.im + b.re};           // A[k] + i conj B[R1 - k]
        u[R1 - k] = cplx<T>{a.re - b.im, b.re - a.im};      // conj A[k] + i B[R1 - k]
    }
}

// W_N^k of a twiddle table (hi and, in single precision, lo part) through the
// constant address space: scalar loads where k is uniform over the wavefront.
template <typename T>
struct TwConst {
    using V = typename Vec2<T>::type;
    const __attribute__((address_space(4))) V* p;
    __device__ __forceinline__ explicit TwConst(const void* t)
        : p((const __attribute__((address_space(4))) V*)t) {}
    __device__ __forceinline__ cplx<T> operator()(int k) const {
        const V v = p[k];
        return {v.x, v.y};
    }
    // x W^k (forward) or x conj(W^k)
    template <bool INV, int N>
    __device__ __forceinline__ cplx<T> mul(cplx<T> x, int k) const {
        const cplx<T> h = (*this)(k);
        if constexpr (std::is_same<T, float>::value) {
            const cplx<T> l = (*this)(N + k);
            return INV ? cmul_split(x, conj(h), conj(l)) : cmul_split(x, h, l);
        } else {
            return INV ? cmulc(x, h) : cmul(x, h);
        }
    }
};

// stockham_level_split with the twiddles from TwConst.
template <class P, int LVL, bool INV, typename T, class Idx>
__device__ __forceinline__ void plane_level(cplx<T>* v, T* lds, const TwConst<T>& tw, int t, Idx idx) {
    constexpr int R = P::radix[LVL];
    constexpr int Ns = P::stride_before(LVL);
    constexpr int NB = P::E / R;
    constexpr int N = P::N;
    if constexpr (LVL > 0) {
        static_for<0, NB * (R - 1)>([&](auto kc) {
            constexpr int b = decltype(kc)::value / (R - 1), r = decltype(kc)::value % (R - 1) + 1;
            const int k = ((t + P::T * b) % Ns) * r * (N / (Ns * R));
            v[b * R + r] = tw.template mul<INV, N>(v[b * R + r], k);
        });
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) dft<R, INV, T>(v + b * R);
    if constexpr (LVL + 1 < P::L) {
        constexpr int R2 = P::radix[LVL + 1];
        constexpr int NB2 = P::E / R2;
#pragma unroll
        for (int part = 0; part < 2; ++part) {
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int j = t + P::T * b;
                const int base = (j / Ns) * Ns * R + (j % Ns);
#pragma unroll
                for (int r = 0; r < R; ++r)
                    lds[idx(base + r * Ns)] = part ? v[b * R + r].im : v[b * R + r].re;
            }
            __syncthreads();
#pragma unroll
            for (int b = 0; b < NB2; ++b) {
                const int j = t + P::T * b;
#pragma unroll
                for (int r = 0; r < R2; ++r) {
                    const T x = lds[idx(j + r * (N / R2))];
                    if (part)
                        v[b * R2 + r].im = x;
                    else
                        v[b * R2 + r].re = x;
                }
            }
            __syncthreads();
        }
        plane_level<P, LVL + 1, INV, T>(v, lds, tw, t, idx);
    }
}

// Group of R1 rows of a z pass: WG threads hold GPW groups.
template <int NZ, int R1>
struct ZRows {
    using FP = typename PlanFor<NZ>::type;
    using IP = Reversed<FP>;
    static constexpr int lanes = R1 * FP::T;
    static constexpr int grow(int g) {
        return lanes * g >= (NZ >= 128 ? 256 : 128) && (lanes * g) % 64 == 0 ? g
               : lanes * g >= 512 ? g : grow(2 * g);
    }
    static constexpr int GPW = lanes >= 192 && lanes % 64 == 0 ? 1 : grow(1);
    static constexpr int PP = R1 * GPW;
    static constexpr int WG = PP * FP::T;
    static constexpr int ROW = NZ + NZ / 16;
    static_assert(WG % 64 == 0, "whole wavefronts");
};

// v[k] *= W_ny^(y0 k) (forward) or its conjugate, k < R1.
template <int R1, bool INV, typename T>
__device__ __forceinline__ void y_twiddle(cplx<T>* v, const void* tw_y, int ny, int y0) {
    const TwConst<T> tw(tw_y);
#pragma unroll
    for (int k = 1; k < R1; ++k) {
        const cplx<T> h = tw(y0 * k);
        if constexpr (std::is_same<T, float>::value) {
            const cplx<T> l = tw(ny + y0 * k);
            v[k] = INV ? cmul_split(v[k], conj(h), conj(l)) : cmul_split(v[k], h, l);
        } else {
            v[k] = INV ? cmulc(v[k], h) : cmul(v[k], h);
        }
    }
}

}  // namespace wdm
