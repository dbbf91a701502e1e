// P2, P4, P6, P8: the passes along y, and plain axis transforms.
#include "passes_common.hpp"

namespace wdm {

bool axis_supported(int n) {
    switch (n) {
        case 16: case 32: case 64: case 96: case 128: case 192: case 256: case 384: case 512:
            return true;
        default:
            return false;
    }
}

bool axis_has_variant(int n) { return axis_supported(n) && has_variant(n); }
bool axis_has_wide(int n) { return axis_supported(n) && has_wide(n); }

// P2 / P4 (psi) and P6 / P8 (half spectrum + Nyquist plane).
template <int NY, typename T, bool INV, bool SPEC, int V>
__global__ __launch_bounds__((wg_size<typename PlanFor<NY, V>::type, T>())) void k_y_fft(
    const MemberDev* __restrict__ mems, int first) {
    using FP = typename PlanFor<NY, V>::type;
    constexpr int PP = pencils_per_wg<FP, T>();
    // P2 / P4 share the machine with the particle kernel: their waves issue
    // first on a SIMD (wave priority 2 of 0-3; the particle waves stay at 0),
    // which keeps these bandwidth-bound passes streaming (256^3 + 1e6 step
    // 0.4079 -> 0.4060 ms on average over four paired runs on two machines)
    if constexpr (!SPEC) __builtin_amdgcn_s_setprio(2);
    __shared__ strided_lds_t<FP, T> lds[lds_entries<FP, T, !SPEC>()];
    __shared__ cplx<T> tw[tw_entries<T>(NY)];
    const MemberDev& m = mems[first + blockIdx.y];
    load_twiddles<NY, wg_size<FP, T>()>(tw, m.tw_y);
    __syncthreads();
    const int64_t nx = m.nx, ny = m.ny, nz = m.nz;
    if constexpr (!SPEC) {
        const Strides sd{nx * nz, nz, ny * nz, nz};
        transform_tile<FP, T, INV, true>(static_cast<cplx<T>*>(m.psi), sd, blockIdx.x, lds, tw);
    } else {
        const int64_t h = nz / 2;
        const int64_t main_tiles = (nx * h + PP - 1) / PP;
        if (int64_t(blockIdx.x) < main_tiles) {
            const Strides sd{nx * h, h, ny * h, h};
            transform_tile<FP, T, INV, true>(static_cast<cplx<T>*>(m.spec), sd, blockIdx.x, lds,
                                             tw);
        } else {
            // kz = nz/2 plane [nx][ny]: y-pencils are contiguous
            const Strides sd{nx, 1, ny, 1};
            transform_tile<FP, T, INV, false>(static_cast<cplx<T>*>(m.spec_nyq), sd,
                                              blockIdx.x - main_tiles, lds, tw);
        }
    }
}


// Plain axis transform of psi or scratch (diagnostics, tests of the FFT), along
// z into z_out if it is given.
template <int N, typename T, bool INV, int AXIS>
__global__ __launch_bounds__((wg_size<typename PlanFor<N>::type, T>())) void k_axis_fft(
    const MemberDev* __restrict__ mems, int first, int which, cplx<T>* __restrict__ z_out) {
    using FP = typename PlanFor<N>::type;
    __shared__ T lds[lds_entries<FP, T, false>()];
    __shared__ cplx<T> tw[tw_entries<T>(N)];
    const MemberDev& m = mems[first + blockIdx.y];
    load_twiddles<N, wg_size<FP, T>()>(tw, AXIS == 0 ? m.tw_x : (AXIS == 1 ? m.tw_y : m.tw_z));
    __syncthreads();
    cplx<T>* data = static_cast<cplx<T>*>(which ? m.scratch : m.psi);
    const int64_t nx = m.nx, ny = m.ny, nz = m.nz;
    if constexpr (AXIS == 2) {
        const Strides sd{nx * ny, 1, nz, 1};
        transform_tile<FP, T, INV, false>(data, sd, blockIdx.x, lds, tw,
                                          z_out != nullptr ? z_out : data);
    } else if constexpr (AXIS == 1) {
        const Strides sd{nx * nz, nz, ny * nz, nz};
        transform_tile<FP, T, INV, true>(data, sd, blockIdx.x, lds, tw);
    } else {
        const Strides sd{ny * nz, ny * nz, 0, ny * nz};
        transform_tile<FP, T, INV, true>(data, sd, blockIdx.x, lds, tw);
    }
}

// Forward z transform into scratch of what SRC names (ZSource), the pencil plan
// and its arithmetic those of k_axis_fft: the copy of psi and the array of the
// contrast (16 and 24 bytes a cell more) are not written.
template <int N, typename T, int SRC>
__global__ __launch_bounds__((wg_size<typename PlanFor<N>::type, T>())) void k_z_fft_from(
    const MemberDev* __restrict__ mems, int first) {
    using FP = typename PlanFor<N>::type;
    using LN = Lanes<FP, T, false>;
    __shared__ T lds[lds_entries<FP, T, false>()];
    __shared__ cplx<T> tw[tw_entries<T>(N)];
    const MemberDev& m = mems[first + blockIdx.y];
    load_twiddles<N, wg_size<FP, T>()>(tw, m.tw_z);
    __syncthreads();
    const LN ln;
    const int64_t rows = int64_t(m.nx) * m.ny;
    const int64_t q = int64_t(blockIdx.x) * LN::PP + ln.p;
    const bool ok = q < rows;
    const int64_t b = ok ? q * N : 0;
    cplx<T> v[FP::E];
    load_slots<FP, FP::first()>(v, static_cast<const cplx<T>*>(m.psi), b, 1, ok, ln);
    if constexpr (SRC == kFromContrast) {
        const double mean = gldr(m.results, 0) / double(rows * N);
#pragma unroll
        for (int s = 0; s < FP::E; ++s) {
            const double r = double(v[s].re) * v[s].re + double(v[s].im) * v[s].im;
            v[s] = cplx<T>{ok ? T(r / mean - 1.0) : T(0), T(0)};
        }
    }
    pencil_fft<FP, false, T>(v, lds, tw, ln.t, ln);
    store_slots<FP, FP::last()>(v, static_cast<cplx<T>*>(m.scratch), b, 1, ok, ln);
}

template <int N>
struct ZFftFrom {
    template <typename T>
    static hipError_t go(const Launch& L, int64_t pencils, int source) {
        dim3 grid(unsigned(tiles<N, T>(pencils)), unsigned(L.count));
        const auto b = block<N, T>();
        if (source == kFromContrast)
            k_z_fft_from<N, T, kFromContrast><<<grid, b, 0, L.stream>>>(L.members, L.first);
        else
            k_z_fft_from<N, T, kFromPsi><<<grid, b, 0, L.stream>>>(L.members, L.first);
        return hipGetLastError();
    }
    static hipError_t run(const Launch& L, int prec, int64_t pencils, int source) {
        return prec ? go<double>(L, pencils, source) : go<float>(L, pencils, source);
    }
};

// Forward transforms of psi that keep only the modes |m| < nc/2 of an axis (zero
// on the coarse Nyquist plane), for the restriction of an N^3 grid: along z from
// psi into scratch [N][N][nc], along y in place into its first nc rows, along x
// into the coarse spectrum out [nc][nc][nc] (in place into the first nc planes where
// out is null), times scale.  A pencil that ends in
// dropped modes is never formed: at 256 -> 128 the three move 350 MB where full
// transforms, the copy of psi and a gather of the kept modes moved 1.1 GB (195 ->
// 67 us).
template <int N, typename T, int AXIS>
__global__ __launch_bounds__((wg_size<typename PlanFor<N>::type, T>())) void k_restrict_fft(
    const MemberDev* __restrict__ mems, int first, int nc, cplx<T>* __restrict__ out, T scale) {
    using FP = typename PlanFor<N>::type;
    constexpr bool STRIDED = AXIS != 2;
    using LN = Lanes<FP, T, STRIDED>;
    __shared__ T lds[lds_entries<FP, T, false>()];
    __shared__ cplx<T> tw[tw_entries<T>(N)];
    const MemberDev& m = mems[first];
    load_twiddles<N, wg_size<FP, T>()>(tw, AXIS == 0 ? m.tw_x : (AXIS == 1 ? m.tw_y : m.tw_z));
    __syncthreads();
    const LN ln;
    const int64_t q = int64_t(blockIdx.x) * LN::PP + ln.p;
    const int64_t plane = int64_t(N) * nc;
    const bool ok = q < (AXIS == 2 ? int64_t(N) * N : AXIS == 1 ? plane : int64_t(nc) * nc);
    const int64_t qq = ok ? q : 0;
    const cplx<T>* in = static_cast<const cplx<T>*>(AXIS == 2 ? m.psi : m.scratch);
    const int64_t b = AXIS == 2 ? qq * N : AXIS == 1 ? qq / nc * plane + qq % nc : qq;
    const int64_t st = AXIS == 2 ? 1 : AXIS == 1 ? nc : plane;
    cplx<T> v[FP::E];
    load_slots<FP, FP::first()>(v, in, b, st, ok, ln);
    pencil_fft<FP, false, T>(v, lds, tw, ln.t, ln);
    if (!ok) return;
    const bool dense = AXIS == 0 && out != nullptr;
    cplx<T>* to = dense ? out : static_cast<cplx<T>*>(m.scratch);
    const int64_t ob = AXIS == 2 ? qq * nc : b, ost = dense ? int64_t(nc) * nc : st;
#pragma unroll
    for (int s = 0; s < FP::E; ++s) {
        const int e = slot_elem<FP, FP::last()>(ln.t, s);
        const int o = e < nc / 2 ? e : e - (N - nc);
        if (e >= nc / 2 && o < nc / 2) continue;
        cplx<T> w = AXIS == 0 ? cscale(v[s], scale) : v[s];
        if (o == nc / 2) w = cplx<T>{T(0), T(0)};
        gst(to, ob + o * ost, w);
    }
}

template <int N>
struct RestrictFft {
    template <typename T>
    static hipError_t go(const Launch& L, int nc, void* out) {
        const auto b = block<N, T>();
        const T scale = T(1.0 / (double(N) * N * N));
        cplx<T>* o = static_cast<cplx<T>*>(out);
        auto g = [](int64_t pencils) { return unsigned(tiles<N, T>(pencils)); };
        k_restrict_fft<N, T, 2><<<g(int64_t(N) * N), b, 0, L.stream>>>(L.members, L.first, nc, o,
                                                                       scale);
        k_restrict_fft<N, T, 1><<<g(int64_t(N) * nc), b, 0, L.stream>>>(L.members, L.first, nc, o,
                                                                        scale);
        k_restrict_fft<N, T, 0><<<g(int64_t(nc) * nc), b, 0, L.stream>>>(L.members, L.first, nc, o,
                                                                         scale);
        return hipGetLastError();
    }
    static hipError_t run(const Launch& L, int prec, int nc, void* out) {
        return prec ? go<double>(L, nc, out) : go<float>(L, nc, out);
    }
};

// Transforms of the vacuum solve's zero-padded grid (Sec. 3.2.1), run on the
// padded member table (doubled lengths, psi = the padded grid).  Only the
// quarter of the padded grid that can be non-zero before the x pass (x < nx,
// y < ny) is read or written along z, and the y passes see the y >= ny half of
// each pencil as zeros (forward) or do not store it (inverse), so the padded
// grid's y >= ny rows are never touched.  The rows hold the modes 0..nz of a real
// row's spectrum, vac_pitch elements apart (all 2 nz of them, 19 + 18 + 11 + 11 us
// for the four and 41 for the x pass at 128^3; now 12 + 12 + 10 + 9 and 28):
//   kVacZFwd  the density rows (real, nz values, held in Phi) zero-extended to
//             2 nz, forward z transform into the padded rows (x < nx, y < ny);
//   kVacYFwd  forward y transform of the x < nx pencils, inputs y >= ny zero;
//   kVacYInv  inverse y transform of the x < nx pencils, outputs y < ny stored;
//   kVacZInv  inverse z transform of the padded rows (x < nx, y < ny), the real
//             part of the first nz values written to Phi.
enum VacMode : int { kVacZFwd = 0, kVacYFwd = 1, kVacYInv = 2, kVacZInv = 3 };

template <int N, typename T, int MODE>
__global__ __launch_bounds__((wg_size<typename PlanFor<N>::type, T>())) void k_vac_fft(
    const MemberDev* __restrict__ mems, int first) {
    using FP = typename PlanFor<N>::type;
    constexpr bool STRIDED = MODE == kVacYFwd || MODE == kVacYInv;
    constexpr bool INV = MODE == kVacYInv || MODE == kVacZInv;
    constexpr int H = N / 2;   // the unpadded length along the transformed axis
    using LN = Lanes<FP, T, STRIDED>;
    __shared__ T lds[lds_entries<FP, T, false>()];
    __shared__ cplx<T> tw[tw_entries<T>(N)];
    const MemberDev& m = mems[first + blockIdx.y];
    load_twiddles<N, wg_size<FP, T>()>(tw, STRIDED ? m.tw_y : m.tw_z);
    __syncthreads();
    const LN ln;
    const int64_t q = int64_t(blockIdx.x) * LN::PP + ln.p;
    cplx<T>* pad = static_cast<cplx<T>*>(m.psi);
    cplx<T> v[FP::E];
    if constexpr (STRIDED) {
        // y pencils of the padded [nx][2ny][pitch] rows: q = x pitch + z, z <= nz
        const int64_t pny = m.ny, pnz = vac_pitch(m.nz);
        const int64_t count = int64_t(m.nx / 2) * pnz;
        const bool ok = q < count && q % pnz <= m.nz / 2;
        const int64_t b = ok ? (q / pnz) * (pny * pnz) + (q % pnz) : 0;
        cplx<T>* lane = pad + (b + int64_t(ln.t) * pnz);
#pragma unroll
        for (int s = 0; s < FP::E; ++s) {
            constexpr int R0 = FP::first();
            const int e = ln.t + slot_const<FP, R0>(s);
            v[s] = (ok && (MODE == kVacYInv || e < H)) ? gld(lane, int64_t(slot_const<FP, R0>(s)) * pnz)
                                                       : cplx<T>{T(0), T(0)};
        }
        pencil_fft<FP, INV, T>(v, lds, tw, ln.t, ln);
        if (!ok) return;
#pragma unroll
        for (int s = 0; s < FP::E; ++s) {
            constexpr int R1 = FP::last();
            const int e = ln.t + slot_const<FP, R1>(s);
            if (MODE == kVacYFwd || e < H) gst(lane, int64_t(slot_const<FP, R1>(s)) * pnz, v[s]);
        }
    } else {
        // rows (x, y), x < nx, y < ny: q = x ny + y
        const int rnx = m.nx / 2, rny = m.ny / 2;
        const bool ok = q < int64_t(rnx) * rny;
        const int64_t x = ok ? q / rny : 0, y = ok ? q - x * rny : 0;
        cplx<T>* row = pad + (x * m.ny + y) * vac_pitch(N);   // padded row
        T* phi = static_cast<T*>(m.phi) + (ok ? q : 0) * H;
        if constexpr (MODE == kVacZFwd) {
#pragma unroll
            for (int s = 0; s < FP::E; ++s) {
                const int e = ln.t + slot_const<FP, FP::first()>(s);
                v[s] = cplx<T>{(ok && e < H) ? gldr(phi, e) : T(0), T(0)};
            }
            pencil_fft<FP, false, T>(v, lds, tw, ln.t, ln);
            if (!ok) return;
#pragma unroll
            for (int s = 0; s < FP::E; ++s) {
                const int e = slot_elem<FP, FP::last()>(ln.t, s);
                if (e <= H) gst(row, e, v[s]);
            }
        } else {
            // the modes above nz are the conjugates of those below
#pragma unroll
            for (int s = 0; s < FP::E; ++s) {
                const int e = slot_elem<FP, FP::first()>(ln.t, s);
                v[s] = ok ? gld(row, e <= H ? e : N - e) : cplx<T>{T(0), T(0)};
                if (e > H) v[s].im = -v[s].im;
            }
            pencil_fft<FP, true, T>(v, lds, tw, ln.t, ln);
            if (!ok) return;
#pragma unroll
            for (int s = 0; s < FP::E; ++s) {
                const int e = ln.t + slot_const<FP, FP::last()>(s);
                if (e < H) gstr(phi, e, v[s].re);
            }
        }
    }
}

template <int N>
struct VacFft {
    template <typename T>
    static hipError_t go(const Launch& L, int64_t pencils, int mode) {
        dim3 grid(unsigned(tiles<N, T>(pencils)), unsigned(L.count));
        const auto b = block<N, T>();
        switch (mode) {
            case kVacZFwd: k_vac_fft<N, T, kVacZFwd><<<grid, b, 0, L.stream>>>(L.members, L.first); break;
            case kVacYFwd: k_vac_fft<N, T, kVacYFwd><<<grid, b, 0, L.stream>>>(L.members, L.first); break;
            case kVacYInv: k_vac_fft<N, T, kVacYInv><<<grid, b, 0, L.stream>>>(L.members, L.first); break;
            default: k_vac_fft<N, T, kVacZInv><<<grid, b, 0, L.stream>>>(L.members, L.first); break;
        }
        return hipGetLastError();
    }
    static hipError_t run(const Launch& L, int prec, int64_t pencils, int mode) {
        return prec ? go<double>(L, pencils, mode) : go<float>(L, pencils, mode);
    }
};

// Spectral kinetic energy: x forward FFT of scratch (already z and y
// transformed) and FP64 partial sums of |k|^2 |psi_k|^2 per work-group.

template <int NY>
struct YFft {
    template <typename T, int V>
    static hipError_t go(const Launch& L, int nx, int nz, bool inv, bool spec) {
        int64_t t;
        if (spec)
            t = tiles<NY, T, V>(int64_t(nx) * (nz / 2)) + tiles<NY, T, V>(nx);
        else
            t = tiles<NY, T, V>(int64_t(nx) * nz);
        dim3 grid(unsigned(t), unsigned(L.count));
        const dim3 b = block<NY, T, V>();
        if (spec) {
            if (inv)
                k_y_fft<NY, T, true, true, V><<<grid, b, 0, L.stream>>>(L.members, L.first);
            else
                k_y_fft<NY, T, false, true, V><<<grid, b, 0, L.stream>>>(L.members, L.first);
        } else {
            if (inv)
                k_y_fft<NY, T, true, false, V><<<grid, b, 0, L.stream>>>(L.members, L.first);
            else
                k_y_fft<NY, T, false, false, V><<<grid, b, 0, L.stream>>>(L.members, L.first);
        }
        return hipGetLastError();
    }
    template <typename T>
    static hipError_t pick(const Launch& L, int nx, int nz, bool inv, bool spec, int var) {
        if constexpr (has_variant(NY))
            if (var == 1) return go<T, 1>(L, nx, nz, inv, spec);
        if constexpr (has_wide(NY)) {
            if (var == 2) return go<T, 2>(L, nx, nz, inv, spec);
            if (var == 3) return go<T, 3>(L, nx, nz, inv, spec);
        }
        return go<T, 0>(L, nx, nz, inv, spec);
    }
    static hipError_t run(const Launch& L, int prec, int nx, int nz, bool inv, bool spec,
                          int var) {
        return prec ? pick<double>(L, nx, nz, inv, spec, var)
                    : pick<float>(L, nx, nz, inv, spec, var);
    }
};

template <int N>
struct AxisFft {
    template <typename T, bool INV>
    static hipError_t go2(const Launch& L, int64_t pencils, int axis, int which, void* z_out) {
        dim3 grid(unsigned(tiles<N, T>(pencils)), unsigned(L.count));
        auto b = block<N, T>();
        cplx<T>* zo = static_cast<cplx<T>*>(z_out);
        if (axis == 0)
            k_axis_fft<N, T, INV, 0><<<grid, b, 0, L.stream>>>(L.members, L.first, which, zo);
        else if (axis == 1)
            k_axis_fft<N, T, INV, 1><<<grid, b, 0, L.stream>>>(L.members, L.first, which, zo);
        else
            k_axis_fft<N, T, INV, 2><<<grid, b, 0, L.stream>>>(L.members, L.first, which, zo);
        return hipGetLastError();
    }
    static hipError_t run(const Launch& L, int prec, int64_t pencils, int axis, bool inv,
                          int which, void* z_out) {
        if (prec)
            return inv ? go2<double, true>(L, pencils, axis, which, z_out)
                       : go2<double, false>(L, pencils, axis, which, z_out);
        return inv ? go2<float, true>(L, pencils, axis, which, z_out)
                   : go2<float, false>(L, pencils, axis, which, z_out);
    }
};

hipError_t launch_y_fft_psi(const Launch& L, int prec, int nx, int ny, int nz, bool inverse,
                            int variant) {
    return dispatch_n<YFft>(ny, L, prec, nx, nz, inverse, false, variant);
}
hipError_t launch_y_fft_spec(const Launch& L, int prec, int nx, int ny, int nz, bool inverse,
                             int variant) {
    return dispatch_n<YFft>(ny, L, prec, nx, nz, inverse, true, variant);
}
hipError_t launch_axis_fft(const Launch& L, int prec, int nx, int ny, int nz, int axis,
                           bool inverse, int which, void* z_out) {
    const int n = axis == 0 ? nx : (axis == 1 ? ny : nz);
    const int64_t pencils = axis == 0 ? int64_t(ny) * nz
                                      : (axis == 1 ? int64_t(nx) * nz : int64_t(nx) * ny);
    return dispatch_n<AxisFft>(n, L, prec, pencils, axis, inverse, which, z_out);
}

hipError_t launch_restrict_fft(const Launch& L, int prec, int nf, int nc, void* out) {
    return dispatch_n<RestrictFft>(nf, L, prec, nc, out);
}

hipError_t launch_z_fft_from(const Launch& L, int prec, int nx, int ny, int nz, int source) {
    return dispatch_n<ZFftFrom>(nz, L, prec, int64_t(nx) * ny, source);
}

hipError_t launch_vac_fft(const Launch& L, int prec, int nx, int ny, int nz, int mode) {
    // nx, ny, nz: the padded lengths
    if (mode == kVacZFwd || mode == kVacZInv)
        return dispatch_n<VacFft>(nz, L, prec, int64_t(nx / 2) * (ny / 2), mode);
    return dispatch_n<VacFft>(ny, L, prec, int64_t(nx / 2) * vac_pitch(nz), mode);
}

int64_t axis_tiles(int n, int64_t pencils, int prec) {
#define WDM_TILES_CASE(N) \
    case N: return prec ? tiles<N, double>(pencils) : tiles<N, float>(pencils);
    switch (n) {
        WDM_TILES_CASE(16)
        WDM_TILES_CASE(32)
        WDM_TILES_CASE(64)
        WDM_TILES_CASE(96)
        WDM_TILES_CASE(128)
        WDM_TILES_CASE(192)
        WDM_TILES_CASE(256)
        WDM_TILES_CASE(384)
        WDM_TILES_CASE(512)
        default: return 0;
    }
#undef WDM_TILES_CASE
}

}  // namespace wdm
