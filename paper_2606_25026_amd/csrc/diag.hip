// Diagnostics of a synchronised state (Sec. 3.6, App. A.1): the paper's
// overall energy terms K, Q, V with the wave momentum, and the radii that
// enclose fixed fractions of the wave mass around a centre node.
#include "wdm_internal.hpp"
#include "fft_device.hpp"

namespace wdm {

constexpr int kDiagFields = 7;   // K, Q, V, Px, Py, Pz, sum |psi|^2 (each times 1/dV)

template <int THREADS>
__device__ __forceinline__ double diag_block_sum(double v, double* red) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = THREADS / 2; w > 0; w >>= 1) {
        if (int(threadIdx.x) < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    const double r = red[0];
    __syncthreads();
    return r;
}

// |psi| and 1 / |psi|^2 in FP64.  From complex64 the square lies between 2^-298
// and 2^257, where the reciprocal square root needs no scaling: Goldschmidt's
// iteration gives both from one, within 2 ulps (zero and infinity apart).
struct Amp {
    double a, inv;
};
template <typename T>
__device__ __forceinline__ Amp amplitude(cplx<T> v) {
    const double rho = double(v.re) * double(v.re) + double(v.im) * double(v.im);
    if constexpr (sizeof(T) == 8) {
        return {sqrt(rho), 1.0 / rho};
    } else {
        const double y = __builtin_amdgcn_rsq(rho);
        double g = rho * y, h = 0.5 * y;
        double r = fma(-h, g, 0.5);
        g = fma(g, r, g);
        h = fma(h, r, h);
        r = fma(-h, g, 0.5);
        g = fma(g, r, g);
        h = fma(h, r, h);
        const double d = fma(-g, g, rho);
        g = fma(d, h, g);
        return {rho == 0.0 || rho == __builtin_inf() ? rho : g, 4.0 * (h * h)};
    }
}

// Per cell, second-order central differences on the periodic nodes:
//   j_a = eta Im(psi* (psi_{+a} - psi_{-a}) / (2 h_a))   (momentum density rho v),
//   K += j.j / (2 rho) for rho > 1e-30,  Q += sum_a ((|psi_{+a}| - |psi_{-a}|) / (2 h_a))^2,
//   V += rho Phi,  P += j,  M += rho.
// A work-group walks an 8 x 64 tile of (y, z) along a range of x: a lane keeps
// its own column's last, current and next values in registers, and the plane's y
// and z neighbours come from LDS; the next plane's loads are in flight while one is
// summed.  Bound by the FP64 instructions of a cell, one after the other: 96 us at
// 256^3 (208 with six neighbours fetched and six square roots a cell; 120 with two
// barriers a plane, a quarter of the range and a divide).
// Fixed ranges, fixed order: deterministic.  The partials go to fields 0..6 and
// are finished by k_reduce_finish.
constexpr int kDiagY = 8, kDiagZ = 64, kDiagThreads = kDiagY * kDiagZ;
template <typename T>
__global__ __launch_bounds__(kDiagThreads) void k_diag_energies(const MemberDev* __restrict__ mems,
                                                                int first, int nblocks) {
    constexpr int LY = kDiagY + 2, LZ = kDiagZ + 2;
    __shared__ double red[kDiagThreads];
    __shared__ cplx<T> planes[2][LY][LZ];   // in turn: one barrier a plane
    __shared__ double amps[2][LY][LZ];
    const MemberDev& m = mems[first];
    const int nx = m.nx, ny = m.ny, nz = m.nz;
    const int64_t nyz = int64_t(ny) * nz;
    const cplx<T>* psi = static_cast<const cplx<T>*>(m.psi);
    const T* phi = static_cast<const T*>(m.phi);
    const double inv2h[3] = {0.5 * m.inv_dx, 0.5 * m.inv_dy, 0.5 * m.inv_dz};
    const double je[3] = {m.eta * inv2h[0], m.eta * inv2h[1], m.eta * inv2h[2]};
    const double qe[3] = {inv2h[0] * inv2h[0], inv2h[1] * inv2h[1], inv2h[2] * inv2h[2]};
    // units of (x range, y tile, z tile), x ranges of at least four planes
    const int ty = (ny + kDiagY - 1) / kDiagY, tz = (nz + kDiagZ - 1) / kDiagZ;
    const int most = min(max(1, nblocks / (ty * tz)), nx / 4);
    const int xl = (nx + most - 1) / most, xs = (nx + xl - 1) / xl;
    const int units = xs * ty * tz;
    const int ly = int(threadIdx.x) / kDiagZ, lz = int(threadIdx.x) % kDiagZ;
    double acc[kDiagFields] = {0, 0, 0, 0, 0, 0, 0};
    for (int unit = blockIdx.x; unit < units; unit += nblocks) {
        const int z0 = (unit % tz) * kDiagZ, y0 = (unit / tz) % ty * kDiagY;
        const int x0 = unit / (tz * ty) * xl, x1 = min(nx, x0 + xl);
        const int y = y0 + ly, z = z0 + lz;
        const bool in = y < ny && z < nz;
        const int64_t own = in ? int64_t(y) * nz + z : 0;
        auto at = [&](int x) { return gld(psi, int64_t(x < 0 ? nx - 1 : x == nx ? 0 : x) * nyz + own); };
        // the halo of the tile's th x tw cells: two rows of y, two columns of z
        const int th = min(kDiagY, ny - y0), tw = min(kDiagZ, nz - z0);
        const int hi = int(threadIdx.x);
        int hy, hz;
        bool halo;
        if (hi < 2 * kDiagZ) {
            hy = hi < kDiagZ ? 0 : th + 1;
            hz = 1 + hi % kDiagZ;
            halo = hz <= tw;
        } else {
            hy = 1 + (hi - 2 * kDiagZ) % kDiagY;
            hz = hi < 2 * kDiagZ + kDiagY ? 0 : tw + 1;
            halo = hy <= th && hi < 2 * kDiagZ + 2 * kDiagY;
        }
        int gy = y0 + hy - 1, gz = z0 + hz - 1;   // -1 .. n: one wrap
        gy = gy < 0 ? ny - 1 : gy == ny ? 0 : gy;
        gz = gz < 0 ? nz - 1 : gz == nz ? 0 : gz;
        const int64_t hat = int64_t(gy) * nz + gz;
        auto halo_at = [&](int x) {
            return halo && x < x1 ? gld(psi, int64_t(x) * nyz + hat) : cplx<T>{T(0), T(0)};
        };
        auto phi_at = [&](int x) {
            return in && x < x1 ? gldr(phi, int64_t(x) * nyz + own) : T(0);
        };
        cplx<T> prev = at(x0 - 1), cur = at(x0), next = at(x0 + 1), hv_next = halo_at(x0);
        T ph_next = phi_at(x0);
        double ap = amplitude<T>(prev).a;
        Amp ac = amplitude<T>(cur);
        for (int x = x0; x < x1; ++x) {
            const cplx<T> after = x + 1 < x1 ? at(x + 2) : cplx<T>{T(0), T(0)};
            const cplx<T> hv = hv_next;
            const T ph = ph_next;
            hv_next = halo_at(x + 1);
            ph_next = phi_at(x + 1);
            const Amp an = amplitude<T>(next);
            auto& sp = planes[x & 1];
            auto& sa = amps[x & 1];
            if (in) {
                sp[ly + 1][lz + 1] = cur;
                sa[ly + 1][lz + 1] = ac.a;
            }
            if (halo) {
                sp[hy][hz] = hv;
                sa[hy][hz] = amplitude<T>(hv).a;
            }
            __syncthreads();
            if (in) {
                const double cr = double(cur.re), ci = double(cur.im);
                const double rho = cr * cr + ci * ci;
                const cplx<T> nb[3][2] = {{next, prev},
                                          {sp[ly + 2][lz + 1], sp[ly][lz + 1]},
                                          {sp[ly + 1][lz + 2], sp[ly + 1][lz]}};
                const double da[3] = {an.a - ap, sa[ly + 2][lz + 1] - sa[ly][lz + 1],
                                      sa[ly + 1][lz + 2] - sa[ly + 1][lz]};
                double j2 = 0.0, q2 = 0.0;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const double dre = double(nb[a][0].re) - double(nb[a][1].re);
                    const double dim = double(nb[a][0].im) - double(nb[a][1].im);
                    const double ja = je[a] * (cr * dim - ci * dre);
                    j2 += ja * ja;
                    acc[3 + a] += ja;
                    q2 += qe[a] * (da[a] * da[a]);
                }
                if (rho > 1e-30) acc[0] += 0.5 * j2 * ac.inv;
                acc[1] += q2;
                acc[2] += rho * double(ph);
                acc[6] += rho;
            }
            prev = cur;
            ap = ac.a;
            cur = next;
            ac = an;
            next = after;
        }
        __syncthreads();   // the next unit's first plane may share this one's buffer
    }
    for (int f = 0; f < kDiagFields; ++f) {
        const double t = diag_block_sum<kDiagThreads>(acc[f], red);
        if (threadIdx.x == 0) m.partials[int64_t(blockIdx.x) * kRedFields + f] = t;
    }
}

// Wave mass per squared node distance s = di^2 + dj^2 + dk^2 (minimum-image
// offsets from the centre node; cubic cells), accumulated with FP64 atomics
// into hist[0..smax] (cleared by the caller).  The cells at offsets (+-a, +-b,
// +-d) share a bin, and with nx = ny so do (a, b) and (b, a): a wavefront takes
// one pair a >= b and sums up to sixteen cells before each atomic addition, which
// is what bounds it: 56 us at 256^3 (one addition a cell: 768).
template <typename T>
__global__ __launch_bounds__(256) void k_radial_hist(const MemberDev* __restrict__ mems, int first,
                                                     int ci, int cj, int ck,
                                                     double* __restrict__ hist) {
    const MemberDev& m = mems[first];
    const int nx = m.nx, ny = m.ny, nz = m.nz;
    const int64_t nyz = int64_t(ny) * nz;
    const int nb = ny / 2 + 1, pairs = (nx / 2 + 1) * nb;
    const int pair = int(blockIdx.x) * 4 + (int(threadIdx.x) >> 6);
    if (pair >= pairs) return;
    const int a = pair / nb, b = pair - a * nb;
    const bool fold = nx == ny;
    if (fold && a < b) return;
    const cplx<T>* psi = static_cast<const cplx<T>*>(m.psi);
    const int lane = int(threadIdx.x) & 63;
    // offsets +-v of an axis: two nodes, or one where they are the same
    auto node = [](int c, int v, int sign, int n) {
        const int i = c + sign * v;
        return i < 0 ? i + n : i >= n ? i - n : i;
    };
    auto twice = [](int v, int n) { return v != 0 && 2 * v != n; };
    const int rows = fold && a != b ? 8 : 4;
    for (int d = lane; d <= nz / 2; d += 64) {
        const int k0 = node(ck, d, 1, nz), k1 = node(ck, d, -1, nz);
        const bool two_k = twice(d, nz);
        // all loads in flight: an image that is no cell of its own reads its
        // partner (or, without the fold, the pair itself) and is left out
        cplx<T> v[8][2];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int va = r < 4 || !fold ? a : b, vb = r < 4 || !fold ? b : a;
            const cplx<T>* row = psi + int64_t(node(ci, va, r & 1 ? -1 : 1, nx)) * nyz +
                                 int64_t(node(cj, vb, r & 2 ? -1 : 1, ny)) * nz;
            v[r][0] = gld(row, k0);
            v[r][1] = gld(row, k1);
        }
        double sum = 0.0;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int va = r < 4 || !fold ? a : b, vb = r < 4 || !fold ? b : a;
            const bool own = r < rows && (!(r & 1) || twice(va, nx)) && (!(r & 2) || twice(vb, ny));
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const double re = double(v[r][k].re), im = double(v[r][k].im);
                sum += own && (k == 0 || two_k) ? re * re + im * im : 0.0;
            }
        }
        if (sum != 0.0) gatomic_add(hist + (a * a + b * b + d * d), sum);
    }
}

// Sums of 1024 bins each; out[f] <- infinity for k_radii_find.
__global__ __launch_bounds__(256) void k_radii_sums(const double* __restrict__ hist, int64_t nbins,
                                                    double* __restrict__ sums,
                                                    double* __restrict__ out) {
    __shared__ double red[256];
    double s = 0.0;
    for (int k = 0; k < 4; ++k) {
        const int64_t i = int64_t(blockIdx.x) * 1024 + k * 256 + threadIdx.x;
        if (i < nbins) s += hist[i];
    }
    const double t = diag_block_sum<256>(s, red);
    if (threadIdx.x == 0) sums[blockIdx.x] = t;
    if (blockIdx.x == 0 && threadIdx.x < 9) out[threadIdx.x] = __builtin_inf();
}

// For f = 0.1, ..., 0.9, the first non-empty bin s whose running sum reaches f
// times the total: out[f] = dx sqrt(s), the smallest over the work-groups (each
// scans 1024 bins behind the sum of those before) by an integer minimum of the
// positive doubles' bit patterns.
__global__ __launch_bounds__(1024) void k_radii_find(const double* __restrict__ hist, int64_t nbins,
                                                     double dx, const double* __restrict__ sums,
                                                     double* __restrict__ out) {
    __shared__ double wsum[16], wbase[16], part[2][16];
    const int tid = int(threadIdx.x), lane = tid & 63, wave = tid >> 6;
    // the sum before this block and the total
    double before = 0.0, all = 0.0;
    for (int b = tid; b < int(gridDim.x); b += 1024) {
        all += sums[b];
        if (b < int(blockIdx.x)) before += sums[b];
    }
    for (int off = 32; off > 0; off >>= 1) {
        all += __shfl_down(all, off);
        before += __shfl_down(before, off);
    }
    if (lane == 0) {
        part[0][wave] = before;
        part[1][wave] = all;
    }
    const int64_t i = int64_t(blockIdx.x) * 1024 + tid;
    const double h = i < nbins ? hist[i] : 0.0;
    double cum = h;
    for (int off = 1; off < 64; off <<= 1) {
        const double o = __shfl_up(cum, off);
        if (lane >= off) cum += o;
    }
    if (lane == 63) wsum[wave] = cum;
    __syncthreads();
    if (tid == 0) {
        double s = 0.0;
        for (int w = 0; w < 16; ++w) s += part[0][w];
        for (int w = 0; w < 16; ++w) {
            wbase[w] = s;
            s += wsum[w];
        }
        s = 0.0;
        for (int w = 0; w < 16; ++w) s += part[1][w];
        part[1][0] = s;
    }
    __syncthreads();
    cum += wbase[wave];
    const double total = part[1][0];
    for (int f = 1; f <= 9; ++f) {
        const double thr = 0.1 * double(f) * total;
        // crossed well before this wavefront (the margin covers the rounding of
        // sums taken in another order): its bins cannot be the first
        if (wbase[wave] * (1.0 - 1e-12) >= thr) continue;
        const unsigned long long hit = __ballot(h > 0.0 && cum >= thr);
        if (hit == 0ull || lane != __ffsll(hit) - 1) continue;
        atomicMin(reinterpret_cast<unsigned long long*>(out) + (f - 1),
                  (unsigned long long)__double_as_longlong(dx * sqrt(double(i))));
    }
}

hipError_t launch_diag_energies(const Launch& L, int prec, int nblocks) {
    if (prec)
        k_diag_energies<double><<<nblocks, kDiagThreads, 0, L.stream>>>(L.members, L.first,
                                                                         nblocks);
    else
        k_diag_energies<float><<<nblocks, kDiagThreads, 0, L.stream>>>(L.members, L.first,
                                                                        nblocks);
    return hipGetLastError();
}

hipError_t launch_mass_radii(const Launch& L, int prec, int nx, int ny, const int centre[3],
                             double dx, double* hist, int64_t nbins, double* sums, double* out) {
    hipError_t e = launch_zero(L.stream, hist, size_t(nbins) * sizeof(double));
    if (e != hipSuccess) return e;
    const unsigned g = unsigned(((nx / 2 + 1) * (ny / 2 + 1) + 3) / 4);
    if (prec)
        k_radial_hist<double><<<g, 256, 0, L.stream>>>(L.members, L.first, centre[0], centre[1],
                                                       centre[2], hist);
    else
        k_radial_hist<float><<<g, 256, 0, L.stream>>>(L.members, L.first, centre[0], centre[1],
                                                      centre[2], hist);
    const unsigned r = unsigned(radii_sums(nbins));
    k_radii_sums<<<r, 256, 0, L.stream>>>(hist, nbins, sums, out);
    k_radii_find<<<r, 1024, 0, L.stream>>>(hist, nbins, dx, sums, out);
    return hipGetLastError();
}

}  // namespace wdm
