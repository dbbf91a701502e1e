// The plane passes of the four-pass step (passes_split.hpp): the radix-R2 part
// of the y transform, the x transform, the factor of each mode and both
// transforms back, in one kernel.  Instantiated for complex64 in
// passes_xy_c64.hip and for complex128 in passes_xy_c128.hip.
#pragma once
#include "passes_split.hpp"

namespace wdm {

enum PlaneOp : int { kPlaneKinetic = 0, kPlaneGreen = 1 };

// OP kPlaneKinetic: psi by the drift factor e_x e_yz / N (FP64 product, rounded
// once, as k_x_kinetic); kPlaneGreen: the half spectrum (column 0 as described
// in passes_split.hpp) by -4 pi G / (|k|^2 N) (as k_x_green).
//
// A work-group's tile is all x, the R2 contiguous rows of one k1 and ZC values
// of z.  A lane loads whole y columns
// (R2 rows at one x and z) straight from memory, so the y radix needs no
// exchange of its own; one exchange turns the columns into x pencils, one
// back.  Neighbouring tiles share 128-byte lines along z and are mapped to
// the same XCD's L2 (mapped round robin, the Green's pass fetched four times its
// bytes).  At 256^3 the kinetic pass takes 70 us in place of 43 + 49 + 43 and the
// Green's pass 40 in place of 25 + 29 + 26: half of it vector instructions, one
// fifth LDS, the rest the load and store phases, which the work-groups of a round
// go through together.  (Persistent work-groups that load the next tile ahead
// were slower, 112 us: the registers cost a third of the wavefronts.)
template <int NX, int R2, int ZC, typename T, int OP>
__global__ __launch_bounds__((PlaneTile<NX, R2, ZC, T>::threads), (PlaneTile<NX, R2, ZC, T>::waves)) void
k_xy_plane(
    const MemberDev* __restrict__ mems, int first) {
    using P = PlaneTile<NX, R2, ZC, T>;
    using FP = typename P::FP;
    using IP = Reversed<FP>;
    constexpr bool KIN = OP == kPlaneKinetic;
    constexpr bool kSplit = std::is_same<T, float>::value;
    // beside the particle kernel its waves issue first, as P2 - P4 do
    if constexpr (KIN) __builtin_amdgcn_s_setprio(2);
    __shared__ T lds[NX * P::LD];
    const MemberDev& m = mems[first + blockIdx.y];
    const int ny = m.ny, nz = m.nz, r1 = ny / R2;
    const int rows = KIN ? nz : nz / 2, per_k1 = rows / ZC;
    // blocks b, b + 8, ... run on one XCD and take neighbouring tiles
    const int tile = int(blockIdx.x & 7) * int(gridDim.x >> 3) + int(blockIdx.x >> 3);
    if (tile >= r1 * per_k1) return;   // uniform
    const int tid = int(threadIdx.x);
    const int k1 = tile / per_k1, z0 = (tile - k1 * per_k1) * ZC;
    // element (x, y0, c) of the tile sits at data + x sx + y0 rows + c (below
    // 2^27 elements: axes of at most 256)
    cplx<T>* data = static_cast<cplx<T>*>(KIN ? m.psi : m.spec) + (k1 * R2 * rows + z0);
    const int sx = ny * rows;
    // y columns of this lane: column q = tid + b threads, c = q % ZC, x = q / ZC
    const int c = tid % ZC;
    static_assert(P::threads % ZC == 0, "a lane's columns share c");
    constexpr int dx = P::threads / ZC;
    const uint32_t at = uint32_t((tid / ZC) * sx + c) * uint32_t(sizeof(cplx<T>));
    cplx<T> u[P::CB][R2];
#pragma unroll
    for (int b = 0; b < P::CB; ++b)
#pragma unroll
        for (int r = 0; r < R2; ++r) u[b][r] = gld_at<true>(data + (b * dx * sx + r * rows), at);
    // x pencil (k2, cc) of this lane, lane t of T
    const int p = tid % P::pencils;
    const int t = P::uniform ? __builtin_amdgcn_readfirstlane(tid / P::pencils) : tid / P::pencils;
    auto idx = [&](int e) { return e * P::LD + p; };
    const int k2 = p / ZC, cc = p % ZC, ky = k1 + r1 * k2;
    // the factors: of the pencil, loaded with the data; of k_x, through the
    // constant address space
    cplx<double> eyz{0.0, 0.0};
    double kyz2 = 0.0;
    T gscale = T(0);
    if constexpr (KIN) {
        const cplx<T>* kin = static_cast<const cplx<T>*>(m.kin);
        constexpr int KS = kSplit ? 2 : 1;
        const int64_t f = KS * (NX + int64_t(ky) * nz + z0 + cc);
        const cplx<T> h = gld(kin, f);
        const cplx<T> l = kSplit ? gld(kin, f + 1) : cplx<T>{T(0), T(0)};
        eyz = cplx<double>{double(h.re) + double(l.re), double(h.im) + double(l.im)};
    } else {
        // column 0 of the k1 > R1/2 rows is the Nyquist plane's
        const int kz = z0 + cc == 0 && 2 * k1 > r1 ? nz / 2 : z0 + cc;
        const double cz = kTwoPi / m.lz;
        const double fy = kTwoPi / m.ly * signed_mode(ky, ny), fz = cz * double(kz);
        kyz2 = fy * fy + fz * fz;
        gscale = T(-m.four_pi_G / (double(m.nx) * double(ny) * double(nz)));
    }
    const TwConst<T> tw(m.tw_x);
    const TwConst<double> ex(m.xtab + NX);
    const __attribute__((address_space(4))) double* kx2 =
        (const __attribute__((address_space(4))) double*)m.xtab;
    // y radix (k1's twiddle was applied by the z pass), columns -> pencils
#pragma unroll
    for (int b = 0; b < P::CB; ++b) dft<R2, false, T>(u[b]);
    cplx<T> v[FP::E];
    const int col = (tid / ZC) * P::LD + c;
#pragma unroll
    for (int part = 0; part < 2; ++part) {
#pragma unroll
        for (int b = 0; b < P::CB; ++b)
#pragma unroll
            for (int r = 0; r < R2; ++r)
                lds[col + b * dx * P::LD + r * ZC] = part ? u[b][r].im : u[b][r].re;
        __syncthreads();
#pragma unroll
        for (int s = 0; s < FP::E; ++s) {
            const T x = lds[idx(slot_elem<FP, FP::first()>(t, s))];
            if (part)
                v[s].im = x;
            else
                v[s].re = x;
        }
        __syncthreads();
    }
    plane_level<FP, 0, false, T>(v, lds, tw, t, idx);
    if constexpr (KIN) {
#pragma unroll
        for (int s = 0; s < FP::E; ++s)
            v[s] = mul64(v[s], cmul(ex(slot_elem<FP, FP::last()>(t, s)), eyz));
    } else {
        auto green = [&](int e, double k2yz) {
            const T k = T(kx2[e] + k2yz);
            return k > T(0) ? gscale * recip(k) : T(0);
        };
        const bool mixed = z0 == 0 && (k1 == 0 || 2 * k1 == r1);
        if (mixed) {
            // column 0 holds A + iB of the kz = 0 and Nyquist planes, both real
            // in x and y: with G the mode at k and G' the one at -k (of this
            // same tile), A = (G + conj G') / 2 and iB = (G - conj G') / 2, so
            // G <- (g + gn) / 2 G + (g - gn) / 2 conj G' with the factors g of A
            // and gn of B.  Pair by pair in LDS, real and imaginary parts in
            // turn, in a loop that keeps the registers of the common path.
            const double cy = kTwoPi / m.ly, cz = kTwoPi / m.lz * double(nz / 2);
#pragma unroll
            for (int part = 0; part < 2; ++part) {
                if (cc == 0) {
#pragma unroll
                    for (int s = 0; s < FP::E; ++s)
                        lds[idx(slot_elem<FP, FP::last()>(t, s))] = part ? v[s].im : v[s].re;
                }
                __syncthreads();
#pragma unroll 1
                for (int i = tid; i < NX * R2; i += P::threads) {
                    const int e = i / R2, k = i % R2;
                    const int em = e == 0 ? 0 : NX - e;
                    const int km = k1 == 0 ? (R2 - k) % R2 : R2 - 1 - k;
                    if (em * R2 + km < i) continue;   // the mirror's lane does both
                    const double fy = cy * signed_mode(k1 + r1 * k, ny);
                    const T g = green(e, fy * fy), gn = green(e, fy * fy + cz * cz);
                    const T p = T(0.5) * (g + gn), q = part ? T(0.5) * (gn - g) : T(0.5) * (g - gn);
                    T* one = lds + e * P::LD + k * ZC;
                    T* two = lds + em * P::LD + km * ZC;
                    const T y = *one, w = *two;
                    *one = p * y + q * w;
                    *two = p * w + q * y;
                }
                __syncthreads();
                if (cc == 0) {
#pragma unroll
                    for (int s = 0; s < FP::E; ++s) {
                        const T y = lds[idx(slot_elem<FP, FP::last()>(t, s))];
                        if (part)
                            v[s].im = y;
                        else
                            v[s].re = y;
                    }
                }
            }
            __syncthreads();
        }
#pragma unroll
        for (int s = 0; s < FP::E; ++s) {
            const T g = green(slot_elem<FP, FP::last()>(t, s), kyz2);
            v[s] = cscale(v[s], mixed && cc == 0 ? T(1) : g);
        }
    }
    plane_level<IP, 0, true, T>(v, lds, tw, t, idx);
    // pencils -> columns, inverse y radix
#pragma unroll
    for (int part = 0; part < 2; ++part) {
#pragma unroll
        for (int s = 0; s < FP::E; ++s)
            lds[idx(slot_elem<IP, IP::last()>(t, s))] = part ? v[s].im : v[s].re;
        __syncthreads();
#pragma unroll
        for (int b = 0; b < P::CB; ++b)
#pragma unroll
            for (int r = 0; r < R2; ++r) {
                const T x = lds[col + b * dx * P::LD + r * ZC];
                if (part)
                    u[b][r].im = x;
                else
                    u[b][r].re = x;
            }
        if (part == 0) __syncthreads();
    }
#pragma unroll
    for (int b = 0; b < P::CB; ++b) dft<R2, true, T>(u[b]);
#pragma unroll
    for (int b = 0; b < P::CB; ++b)
#pragma unroll
        for (int r = 0; r < R2; ++r) gst_at<true>(data + (b * dx * sx + r * rows), at, u[b][r]);
}

template <typename T, int OP>
struct XyLaunch {
    template <int NX, int R2, int ZC>
    static hipError_t go(const Launch& L, int ny, int nz) {
        using P = PlaneTile<NX, R2, ZC, T>;
        const int r1 = ny / R2;
        int64_t g = int64_t(r1) * ((OP == kPlaneKinetic ? nz : nz / 2) / ZC);
        g = (g + 7) / 8 * 8;   // the kernel's tile order takes a multiple of the eight XCDs
        k_xy_plane<NX, R2, ZC, T, OP><<<dim3(unsigned(g), unsigned(L.count)), P::threads, 0, L.stream>>>(
            L.members, L.first);
        return hipGetLastError();
    }
    template <int NX>
    static hipError_t with_r2(const Launch& L, int ny, int nz) {
        switch (ny / y_radix(ny)) {
            case 4:
                return plane_zc(4, nz) == 16 ? go<NX, 4, 16>(L, ny, nz) : go<NX, 4, 8>(L, ny, nz);
            case 8: return go<NX, 8, plane_zc(8, 16)>(L, ny, nz);
            case 16: return go<NX, 16, plane_zc(16, 16)>(L, ny, nz);
            default: return hipErrorInvalidValue;
        }
    }
    static hipError_t run(const Launch& L, int nx, int ny, int nz) {
        if (y_radix(ny) == 0) return hipErrorInvalidValue;
        switch (nx) {
            case 16: return with_r2<16>(L, ny, nz);
            case 32: return with_r2<32>(L, ny, nz);
            case 64: return with_r2<64>(L, ny, nz);
            case 96: return with_r2<96>(L, ny, nz);
            case 128: return with_r2<128>(L, ny, nz);
            case 192: return with_r2<192>(L, ny, nz);
            case 256: return with_r2<256>(L, ny, nz);
            default: return hipErrorInvalidValue;
        }
    }
};

}  // namespace wdm
