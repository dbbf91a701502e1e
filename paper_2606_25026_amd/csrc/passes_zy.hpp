// The z passes of the four-pass step (passes_split.hpp): P1 and P5 with the
// radix-R1 part of the y transform.  Instantiated for complex64 in
// passes_zy_c64.hip and for complex128 in passes_zy_c128.hip.
//
// A work-group holds its rows in two layouts: "pencils" (a lane has E values of
// one row; loads, stores and the z transform) and "columns" (a lane has the R1
// rows' values at one z; the y radix, and loads and stores of the (y0, k1)
// form, whose lanes run along z).  An LDS exchange turns one into the other.
// P1 moves 24 bytes per cell (20 where no particle needs Phi) and P5 24; at 256^3
// P1 takes 80 us (its vector units two thirds busy, its LDS a third) and P5 60
// without particles.  Every transform and exchange below ends with a barrier after
// its last LDS read, so the next one may write at once.
#pragma once
#include "passes_split.hpp"

namespace wdm {

// Whether a z pass exchanges real and imaginary parts in turn.  Whole values
// (half the barriers and LDS instructions) in single precision, where four
// work-groups still fit a CU, as many as the registers allow: 246 against 251 us
// a 256^3 step; in double precision they would be two.
template <class FP, typename T>
constexpr bool zy_split() {
    return sizeof(T) == 8 && split_exchange<FP, false>();
}

// Work-group coordinates of a z pass.
template <int NZ, int R1>
struct ZCoord {
    using Z = ZRows<NZ, R1>;
    int t, p;             // pencil layout: lane of the pencil, pencil
    int r2, ny;
    int64_t g0;           // first group
    __device__ __forceinline__ explicit ZCoord(const MemberDev& m) {
        t = int(threadIdx.x) % Z::FP::T;
        p = int(threadIdx.x) / Z::FP::T;
        ny = m.ny;
        r2 = m.ny / R1;
        g0 = int64_t(blockIdx.x) * Z::GPW;
    }
    // first row (x ny + y0) of group g of the work-group, and its y0
    __device__ __forceinline__ int64_t row0(int g, int& y0) const {
        const int64_t G = g0 + g;
        const int64_t x = G / r2;
        y0 = int(G - x * r2);
        return x * ny + y0;
    }
    // this lane's pencil row
    __device__ __forceinline__ int64_t row() const {
        int y0;
        const int64_t r = row0(p / R1, y0);
        return r + int64_t(p % R1) * r2;
    }
    // LDS slot of element e of pencil q
    __device__ __forceinline__ static int slot(int q, int e) { return q * Z::ROW + e + (e >> 4); }
    // pencil layout's slot
    __device__ __forceinline__ int operator()(int e) const { return slot(p, e); }
};

// Columns of width NC (NZ, or NZ/2 of a half spectrum) over the work-group:
// this lane's column number i is tid + i WG.
template <int NZ, int R1, int NC>
struct ZCols {
    using Z = ZRows<NZ, R1>;
    static constexpr int total = Z::GPW * NC;
    static constexpr int per = (total + Z::WG - 1) / Z::WG;
    __device__ __forceinline__ static bool active(int i) {
        return total % Z::WG == 0 || int(threadIdx.x) + i * Z::WG < total;
    }
    // (0 of one group: the row addresses are then uniform)
    __device__ __forceinline__ static int group(int i) {
        return Z::GPW == 1 ? 0 : (int(threadIdx.x) + i * Z::WG) / NC;
    }
    __device__ __forceinline__ static int kz(int i) {
        return int(threadIdx.x) + i * Z::WG - group(i) * NC;
    }
    // byte offset of kz in a row
    template <typename T>
    __device__ __forceinline__ static uint32_t at(int i) {
        return uint32_t(kz(i)) * uint32_t(sizeof(cplx<T>));
    }
};

// y0 of a column's group.  The groups of a wavefront are one where the column
// width is a multiple of 64: the twiddles' addresses are then uniform.
template <int NC>
__device__ __forceinline__ int uniform_y0(int y0) {
    if constexpr (NC % 64 == 0)
        return __builtin_amdgcn_readfirstlane(y0);
    else
        return y0;
}

// ===========================================================================
// P1: half spectrum -> (y radix inverse, Hermitian completion, z inverse) Phi,
// kick of psi, z transform and y radix of psi.
// ===========================================================================
template <int NZ, int R1, typename T, int OP, bool GEN>
__global__ __launch_bounds__((ZRows<NZ, R1>::WG)) void k_zy_potential_kick(
    const MemberDev* __restrict__ mems, int first, int full) {
    using Z = ZRows<NZ, R1>;
    using FP = typename Z::FP;
    using IP = typename Z::IP;
    constexpr bool SPLIT = zy_split<FP, T>();
    using LT = std::conditional_t<SPLIT, T, cplx<T>>;
    constexpr int H = NZ / 2;
    constexpr bool MASK = GEN && OP != kZPhiOnly;
    __shared__ LT lds[Z::PP * Z::ROW];
    __shared__ cplx<T> tw[tw_entries<T>(NZ)];
    __shared__ double bz[MASK ? NZ : 1];
    const MemberDev& m = mems[first + blockIdx.y];
    const ZCoord<NZ, R1> zc(m);
    const int64_t row = zc.row();
    load_twiddles<NZ, Z::WG>(tw, m.tw_z);
    // the absorbing boundary follows the merged and the closing kick, not the
    // opening one
    const bool mask = MASK && (OP == kZKickOnly || full);
    double bxy = 1.0;
    if constexpr (MASK) {
        if (mask) bxy = load_absorb<NZ, Z::WG>(bz, m, row, true);
    }
    // psi and the spectrum columns are loaded together: one memory wait
    cplx<T>* psi = static_cast<cplx<T>*>(m.psi);
    cplx<T> w[OP == kZPhiOnly ? 1 : FP::E];
    if constexpr (OP != kZPhiOnly) load_slots<FP, FP::first()>(w, psi, row * NZ, 1, true, zc);
    using HC = ZCols<NZ, R1, H>;
    cplx<T> u[HC::per][R1];
    int yy[HC::per];
#pragma unroll
    for (int i = 0; i < HC::per; ++i) {
        if (!HC::active(i)) continue;
        const int64_t r0 = zc.row0(HC::group(i), yy[i]);
        const cplx<T>* s = static_cast<const cplx<T>*>(m.spec) + r0 * H;
#pragma unroll
        for (int k = 0; k < R1; ++k) u[i][k] = gld_at<Z::GPW == 1>(s + k * zc.r2 * H, HC::template at<T>(i));
    }
#pragma unroll
    for (int i = 0; i < HC::per; ++i) {
        if (!HC::active(i)) continue;
        y_twiddle<R1, true, T>(u[i], m.tw_y, zc.ny, uniform_y0<H>(yy[i]));
        // the kz = 0 and kz = NZ/2 values of a row are both real once y is back
        // in real space: column 0 carries a0 + i aH through the y radix
        if (HC::kz(i) == 0) unpack_column0<R1, T>(u[i]);
        dft<R1, true, T>(u[i]);
    }
    // columns -> Hermitian-completed pencils in the inverse plan's input layout
    cplx<T> v[FP::E];
    if constexpr (SPLIT) {
#pragma unroll
        for (int part = 0; part < 2; ++part) {
#pragma unroll
            for (int i = 0; i < HC::per; ++i) {
                if (!HC::active(i)) continue;
                const int kz = HC::kz(i), q0 = HC::group(i) * R1;
#pragma unroll
                for (int j = 0; j < R1; ++j) {
                    const T x = part ? (kz == 0 ? T(0) : u[i][j].im) : u[i][j].re;
                    lds[zc.slot(q0 + j, kz)] = x;
                    if (kz == 0) lds[zc.slot(q0 + j, H)] = part ? T(0) : u[i][j].im;
                }
            }
            __syncthreads();
#pragma unroll
            for (int s = 0; s < FP::E; ++s) {
                const int e = slot_elem<IP, IP::first()>(zc.t, s);
                const T x = e <= H ? lds[zc(e)] : lds[zc(NZ - e)];
                if (part)
                    v[s].im = e <= H ? x : -x;
                else
                    v[s].re = x;
            }
            __syncthreads();
        }
    } else {
#pragma unroll
        for (int i = 0; i < HC::per; ++i) {
            if (!HC::active(i)) continue;
            const int kz = HC::kz(i), q0 = HC::group(i) * R1;
#pragma unroll
            for (int j = 0; j < R1; ++j) {
                lds[zc.slot(q0 + j, kz)] = kz == 0 ? cplx<T>{u[i][j].re, T(0)} : u[i][j];
                if (kz == 0) lds[zc.slot(q0 + j, H)] = cplx<T>{u[i][j].im, T(0)};
            }
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < FP::E; ++s) {
            const int e = slot_elem<IP, IP::first()>(zc.t, s);
            v[s] = e <= H ? lds[zc(e)] : conj(lds[zc(NZ - e)]);
        }
        __syncthreads();
    }
    pencil_fft<IP, true, T>(v, lds, tw, zc.t, zc);
    T phi[FP::E];
    T* gphi = static_cast<T*>(m.phi) + row * NZ;
#pragma unroll
    for (int s = 0; s < FP::E; ++s) phi[s] = v[s].re;
    if constexpr (GEN) {
        if (m.ext != nullptr) {
            const T* ge = static_cast<const T*>(m.ext) + row * NZ;
#pragma unroll
            for (int s = 0; s < FP::E; ++s) phi[s] += gldr(ge, slot_elem<FP, FP::first()>(zc.t, s));
        }
    }
    if (OP != kZKickFft || phi_wanted(m)) {
#pragma unroll
        for (int s = 0; s < FP::E; ++s) gstr(gphi, slot_elem<FP, FP::first()>(zc.t, s), phi[s]);
    }
    watch_max<FP::E>(m.watch, m.watch_n, phi);
    if constexpr (OP == kZPhiOnly) return;
    const double dt = gldr(m.dt, 0);
    const double c = -(full ? dt : 0.5 * dt) / m.eta;
    if constexpr (GEN) {
        if (m.kappa != 0.0) {
            T r2[FP::E];
#pragma unroll
            for (int s = 0; s < FP::E; ++s) r2[s] = w[s].re * w[s].re + w[s].im * w[s].im;
            watch_max<FP::E>(m.watch + m.watch_n, m.watch_n, r2);
        }
        kick_general<FP, T>(v, w, phi, m, mask, full != 0, bxy, bz, c, zc);
    } else {
#pragma unroll
        for (int s = 0; s < FP::E; ++s) v[s] = rotate(w[s], double(phi[s]) * c);
    }
    if constexpr (OP == kZKickOnly) {
        store_slots<FP, FP::first()>(v, psi, row * NZ, 1, true, zc);
        return;
    }
    pencil_fft<FP, false, T>(v, lds, tw, zc.t, zc);
    // pencils -> columns, y radix, store in the (y0, k1) form
    using WC = ZCols<NZ, R1, NZ>;
    cplx<T> c2[WC::per][R1];
    if constexpr (SPLIT) {
#pragma unroll
        for (int part = 0; part < 2; ++part) {
#pragma unroll
            for (int s = 0; s < FP::E; ++s)
                lds[zc(slot_elem<FP, FP::last()>(zc.t, s))] = part ? v[s].im : v[s].re;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < WC::per; ++i) {
                if (!WC::active(i)) continue;
#pragma unroll
                for (int j = 0; j < R1; ++j) {
                    const T x = lds[zc.slot(WC::group(i) * R1 + j, WC::kz(i))];
                    if (part)
                        c2[i][j].im = x;
                    else
                        c2[i][j].re = x;
                }
            }
            if (part == 0) __syncthreads();
        }
    } else {
#pragma unroll
        for (int s = 0; s < FP::E; ++s) lds[zc(slot_elem<FP, FP::last()>(zc.t, s))] = v[s];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < WC::per; ++i) {
            if (!WC::active(i)) continue;
#pragma unroll
            for (int j = 0; j < R1; ++j) c2[i][j] = lds[zc.slot(WC::group(i) * R1 + j, WC::kz(i))];
        }
    }
#pragma unroll
    for (int i = 0; i < WC::per; ++i) {
        if (!WC::active(i)) continue;
        int y0;
        const int64_t r0 = zc.row0(WC::group(i), y0);
        dft<R1, false, T>(c2[i]);
        y_twiddle<R1, false, T>(c2[i], m.tw_y, zc.ny, uniform_y0<NZ>(y0));
        cplx<T>* d = psi + r0 * NZ;
#pragma unroll
        for (int k = 0; k < R1; ++k) gst_at<Z::GPW == 1>(d + k * zc.r2 * NZ, WC::template at<T>(i), c2[i][k]);
    }
}

// ===========================================================================
// P5: y radix and z inverse of psi (kDensInvFft) or psi in real space
// (kDensDirect), density, z transform and y radix of the half spectrum.
// `keep` and `scal` as in k_z_density.
// ===========================================================================
template <int NZ, int R1, typename T, int OP>
__global__ __launch_bounds__((ZRows<NZ, R1>::WG)) void k_zy_density(
    const MemberDev* __restrict__ mems, int first, int keep, const double* __restrict__ scal) {
    using Z = ZRows<NZ, R1>;
    using FP = typename Z::FP;
    using IP = typename Z::IP;
    constexpr bool SPLIT = zy_split<FP, T>();
    using LT = std::conditional_t<SPLIT, T, cplx<T>>;
    constexpr int H = NZ / 2;
    __shared__ LT lds[Z::PP * Z::ROW];
    __shared__ cplx<T> tw[tw_entries<T>(NZ)];
    const MemberDev& m = mems[first + blockIdx.y];
    const ZCoord<NZ, R1> zc(m);
    const int64_t row = zc.row();
    load_twiddles<NZ, Z::WG>(tw, m.tw_z);
    cplx<T>* psi = static_cast<cplx<T>*>(m.psi);
    cplx<T> v[FP::E];
    if constexpr (OP == kDensInvFft) {
        using WC = ZCols<NZ, R1, NZ>;
        cplx<T> u[WC::per][R1];
        int yy[WC::per];
#pragma unroll
        for (int i = 0; i < WC::per; ++i) {
            if (!WC::active(i)) continue;
            const int64_t r0 = zc.row0(WC::group(i), yy[i]);
            const cplx<T>* s = psi + r0 * NZ;
#pragma unroll
            for (int k = 0; k < R1; ++k) u[i][k] = gld_at<Z::GPW == 1>(s + k * zc.r2 * NZ, WC::template at<T>(i));
        }
#pragma unroll
        for (int i = 0; i < WC::per; ++i) {
            if (!WC::active(i)) continue;
            y_twiddle<R1, true, T>(u[i], m.tw_y, zc.ny, uniform_y0<NZ>(yy[i]));
            dft<R1, true, T>(u[i]);
        }
        // columns -> pencils
#pragma unroll
        for (int part = 0; part < (SPLIT ? 2 : 1); ++part) {
#pragma unroll
            for (int i = 0; i < WC::per; ++i) {
                if (!WC::active(i)) continue;
#pragma unroll
                for (int j = 0; j < R1; ++j) {
                    const int at = zc.slot(WC::group(i) * R1 + j, WC::kz(i));
                    if constexpr (SPLIT)
                        lds[at] = part ? u[i][j].im : u[i][j].re;
                    else
                        lds[at] = u[i][j];
                }
            }
            __syncthreads();
#pragma unroll
            for (int s = 0; s < FP::E; ++s) {
                const int e = slot_elem<IP, IP::first()>(zc.t, s);
                if constexpr (!SPLIT)
                    v[s] = lds[zc(e)];
                else if (part)
                    v[s].im = lds[zc(e)];
                else
                    v[s].re = lds[zc(e)];
            }
            __syncthreads();
        }
        pencil_fft<IP, true, T>(v, lds, tw, zc.t, zc);
        store_slots<FP, FP::first()>(v, psi, row * NZ, 1, true, zc);
    } else {
        load_slots<FP, FP::first()>(v, psi, row * NZ, 1, true, zc);
        if (scal != nullptr) {
            const double a = gldr(scal, 2);
            const T f = a > 0.0 ? T(sqrt(gldr(scal, 1) / a)) : T(1);
#pragma unroll
            for (int s = 0; s < FP::E; ++s) v[s] = cplx<T>{v[s].re * f, v[s].im * f};
            store_slots<FP, FP::first()>(v, psi, row * NZ, 1, true, zc);
        }
    }
    // rho = |psi|^2 + rho_b; a member without particles has no rho_b to read
    // or clear, a static or kept deposit stays
    T* rb = static_cast<T*>(m.rho_b) + row * NZ + zc.t;
    const bool touched = m.np > 0;
    const bool clear = touched && !m.static_baryons && first + int(blockIdx.y) != keep;
    T rbv[FP::E];
#pragma unroll
    for (int s = 0; s < FP::E; ++s)
        rbv[s] = touched ? gldr(rb, slot_const<FP, FP::first()>(s)) : T(0);
#pragma unroll
    for (int s = 0; s < FP::E; ++s) {
        v[s] = cplx<T>{v[s].re * v[s].re + v[s].im * v[s].im + rbv[s], T(0)};
        // (most of a grid holds no baryons: 4 bytes a cell not written)
        if (clear && rbv[s] != T(0)) gstr(rb, slot_const<FP, FP::first()>(s), T(0));
    }
    pencil_fft<FP, false, T>(v, lds, tw, zc.t, zc);
    // pencils -> columns of the half spectrum.  The density is real, so the
    // kz = 0 and kz = NZ/2 values are too: column 0 carries F0 + i FH.
    using HC = ZCols<NZ, R1, H>;
    cplx<T> u[HC::per][R1];
#pragma unroll
    for (int part = 0; part < (SPLIT ? 2 : 1); ++part) {
#pragma unroll
        for (int s = 0; s < FP::E; ++s) {
            const int e = slot_elem<FP, FP::last()>(zc.t, s);
            if constexpr (SPLIT) {
                if (part == 0) {
                    if (e < H) lds[zc(e)] = v[s].re;
                } else {
                    if (e > 0 && e < H) lds[zc(e)] = v[s].im;
                    if (e == H) lds[zc(0)] = v[s].re;
                }
            } else {
                if (e > 0 && e < H) lds[zc(e)] = v[s];
                if (e == 0) lds[zc(0)].re = v[s].re;
                if (e == H) lds[zc(0)].im = v[s].re;
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < HC::per; ++i) {
            if (!HC::active(i)) continue;
#pragma unroll
            for (int j = 0; j < R1; ++j) {
                const int at = zc.slot(HC::group(i) * R1 + j, HC::kz(i));
                if constexpr (!SPLIT)
                    u[i][j] = lds[at];
                else if (part)
                    u[i][j].im = lds[at];
                else
                    u[i][j].re = lds[at];
            }
        }
        if (SPLIT && part == 0) __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < HC::per; ++i) {
        if (!HC::active(i)) continue;
        int y0;
        const int64_t r0 = zc.row0(HC::group(i), y0);
        dft<R1, false, T>(u[i]);
        if (HC::kz(i) == 0) pack_column0<R1, T>(u[i]);
        y_twiddle<R1, false, T>(u[i], m.tw_y, zc.ny, uniform_y0<H>(y0));
        cplx<T>* d = static_cast<cplx<T>*>(m.spec) + r0 * H;
#pragma unroll
        for (int k = 0; k < R1; ++k) gst_at<Z::GPW == 1>(d + k * zc.r2 * H, HC::template at<T>(i), u[i][k]);
    }
}

// The half spectrum's rows from real space in y to the (y0, k1) form (scaled
// by 1 / R1, so that P1's inverse radix restores them), or back; column 0 with
// the Nyquist plane, of whose values in real space the real parts count.  One
// column (x, y0, kz) per lane.
template <int R1, typename T>
__global__ __launch_bounds__(256) void k_spec_form(const MemberDev* __restrict__ mems, int first,
                                                   int to_split) {
    const MemberDev& m = mems[first + blockIdx.y];
    const int h = m.nz / 2, r2 = m.ny / R1;
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    const int64_t G = i / h;
    const int kz = int(i - G * h);
    if (G >= int64_t(m.nx) * r2) return;
    const int64_t x = G / r2;
    const int y0 = int(G - x * r2);
    const int64_t row = x * m.ny + y0;
    cplx<T>* s = static_cast<cplx<T>*>(m.spec) + row * h + kz;
    cplx<T>* q = static_cast<cplx<T>*>(m.spec_nyq) + row;
    cplx<T> v[R1];
#pragma unroll
    for (int k = 0; k < R1; ++k) v[k] = gld(s, int64_t(k) * r2 * h);
    if (to_split) {
        if (kz == 0) {
#pragma unroll
            for (int k = 0; k < R1; ++k) v[k].im = gld(q, int64_t(k) * r2).re;
        }
        dft<R1, false, T>(v);
        if (kz == 0) pack_column0<R1, T>(v);
        y_twiddle<R1, false, T>(v, m.tw_y, m.ny, y0);
    } else {
        y_twiddle<R1, true, T>(v, m.tw_y, m.ny, y0);
        if (kz == 0) unpack_column0<R1, T>(v);
        dft<R1, true, T>(v);
        if (kz == 0) {
#pragma unroll
            for (int k = 0; k < R1; ++k) {
                gst(q, int64_t(k) * r2, cplx<T>{v[k].im, T(0)});
                v[k].im = T(0);
            }
        }
    }
    const T f = to_split ? T(1.0 / R1) : T(1);
#pragma unroll
    for (int k = 0; k < R1; ++k) gst(s, int64_t(k) * r2 * h, cscale(v[k], f));
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <typename T>
struct ZyLaunch {
    template <int R1>
    static hipError_t form_go(const Launch& L, int nx, int ny, int nz, bool to_split) {
        const int64_t n = int64_t(nx) * (ny / R1) * (nz / 2);
        k_spec_form<R1, T><<<dim3(unsigned((n + 255) / 256), unsigned(L.count)), 256, 0, L.stream>>>(
            L.members, L.first, to_split ? 1 : 0);
        return hipGetLastError();
    }
    static hipError_t form(const Launch& L, int nx, int ny, int nz, bool to_split) {
        switch (y_radix(ny)) {
            case 4: return form_go<4>(L, nx, ny, nz, to_split);
            case 8: return form_go<8>(L, nx, ny, nz, to_split);
            case 12: return form_go<12>(L, nx, ny, nz, to_split);
            case 16: return form_go<16>(L, nx, ny, nz, to_split);
            default: return hipErrorInvalidValue;
        }
    }
    template <int NZ, int R1>
    static dim3 grid(const Launch& L, int nx, int ny) {
        return dim3(unsigned(int64_t(nx) * (ny / R1) / ZRows<NZ, R1>::GPW), unsigned(L.count));
    }
    template <int NZ, int R1>
    static hipError_t kick_go(const Launch& L, int nx, int ny, ZOp op, KickMode k, bool gen) {
        const dim3 g = grid<NZ, R1>(L, nx, ny), b(ZRows<NZ, R1>::WG);
        const int full = k == kFullKick ? 1 : 0;
        if (gen) {
            if (op == kZPhiOnly)
                k_zy_potential_kick<NZ, R1, T, kZPhiOnly, true><<<g, b, 0, L.stream>>>(L.members, L.first, full);
            else if (op == kZKickOnly)
                k_zy_potential_kick<NZ, R1, T, kZKickOnly, true><<<g, b, 0, L.stream>>>(L.members, L.first, full);
            else
                k_zy_potential_kick<NZ, R1, T, kZKickFft, true><<<g, b, 0, L.stream>>>(L.members, L.first, full);
        } else {
            if (op == kZPhiOnly)
                k_zy_potential_kick<NZ, R1, T, kZPhiOnly, false><<<g, b, 0, L.stream>>>(L.members, L.first, full);
            else if (op == kZKickOnly)
                k_zy_potential_kick<NZ, R1, T, kZKickOnly, false><<<g, b, 0, L.stream>>>(L.members, L.first, full);
            else
                k_zy_potential_kick<NZ, R1, T, kZKickFft, false><<<g, b, 0, L.stream>>>(L.members, L.first, full);
        }
        return hipGetLastError();
    }
    template <int NZ, int R1>
    static hipError_t dens_go(const Launch& L, int nx, int ny, DensOp op, int keep, const double* scal) {
        const dim3 g = grid<NZ, R1>(L, nx, ny), b(ZRows<NZ, R1>::WG);
        if (op == kDensDirect)
            k_zy_density<NZ, R1, T, kDensDirect><<<g, b, 0, L.stream>>>(L.members, L.first, keep, scal);
        else if (op == kDensInvFft && scal == nullptr)
            k_zy_density<NZ, R1, T, kDensInvFft><<<g, b, 0, L.stream>>>(L.members, L.first, keep, scal);
        else
            return hipErrorInvalidValue;
        return hipGetLastError();
    }
    // F::template go<NZ, R1>() for the run-time pair
    template <int NZ, class F>
    static hipError_t with_r1(int r1, F&& f) {
        if constexpr (zrows_supported(NZ, 4))
            if (r1 == 4) return f(std::integral_constant<int, NZ>{}, std::integral_constant<int, 4>{});
        if constexpr (zrows_supported(NZ, 8))
            if (r1 == 8) return f(std::integral_constant<int, NZ>{}, std::integral_constant<int, 8>{});
        if constexpr (zrows_supported(NZ, 12))
            if (r1 == 12) return f(std::integral_constant<int, NZ>{}, std::integral_constant<int, 12>{});
        if constexpr (zrows_supported(NZ, 16))
            if (r1 == 16) return f(std::integral_constant<int, NZ>{}, std::integral_constant<int, 16>{});
        return hipErrorInvalidValue;
    }
    template <class F>
    static hipError_t with(int nz, int r1, F&& f) {
        switch (nz) {
            case 16: return with_r1<16>(r1, f);
            case 32: return with_r1<32>(r1, f);
            case 64: return with_r1<64>(r1, f);
            case 96: return with_r1<96>(r1, f);
            case 128: return with_r1<128>(r1, f);
            case 192: return with_r1<192>(r1, f);
            case 256: return with_r1<256>(r1, f);
            default: return hipErrorInvalidValue;
        }
    }
    static hipError_t kick(const Launch& L, int nx, int ny, int nz, ZOp op, KickMode k, bool gen) {
        return with(nz, y_radix(ny), [&](auto n, auto r) {
            return kick_go<decltype(n)::value, decltype(r)::value>(L, nx, ny, op, k, gen);
        });
    }
    static hipError_t density(const Launch& L, int nx, int ny, int nz, DensOp op, int keep,
                              const double* scal) {
        return with(nz, y_radix(ny), [&](auto n, auto r) {
            return dens_go<decltype(n)::value, decltype(r)::value>(L, nx, ny, op, keep, scal);
        });
    }
};

}  // namespace wdm
