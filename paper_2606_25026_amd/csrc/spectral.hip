// Spectral utilities of the learned-corrector workload: the shell power spectrum
// of the density contrast and the distance between two fields.
#include <algorithm>

#include "wdm_internal.hpp"
#include "fft_device.hpp"

namespace wdm {

// Shell sums of |delta_k|^2 / N^2 over b = round(|m|) < nbins (cubic grid);
// each work-group writes part[block][0..nbins) sums and [nbins..2 nbins) counts.
// The modes (+-a, +-b, +-d) and (+-b, +-a, +-d) share a shell: a wavefront takes
// pairs a >= b and a lane one d, which sums up to sixteen modes before its two
// LDS additions.  Bound by its reads of the spectrum: 18 us at 256^3 (two
// additions a mode over 64 work-groups: 565).
constexpr int kPkMaxBins = 1024;
constexpr int kPkDoubles = 64 * 2 * kPkMaxBins;   // partials of all work-groups
constexpr int kPkMaxBlocks = 1024;

// Work-groups of an n^3 grid: as many as the partials hold, at most one per four
// pairs (a, b).  Each one's partials are a further term of the finishing sum: the
// whole spectrum of one or eight bins takes 56, 57 and 62 us at 16^3, 32^3 and 64^3,
// 73-79 with 1024 work-groups.
static int shell_blocks(int n, int nbins) {
    const int nh = n / 2 + 1;
    return std::min({kPkMaxBlocks, kPkDoubles / (2 * nbins), (nh * nh + 3) / 4});
}

template <typename T>
__global__ __launch_bounds__(256) void k_shells(const MemberDev* __restrict__ mems, int first,
                                                int nbins, double* __restrict__ part) {
    __shared__ double sum[kPkMaxBins];
    __shared__ unsigned long long cnt[kPkMaxBins];
    const MemberDev& m = mems[first];
    for (int b = int(threadIdx.x); b < nbins; b += 256) {
        sum[b] = 0.0;
        cnt[b] = 0ull;
    }
    __syncthreads();
    const int n = m.nx, nh = n / 2 + 1;
    const double N = double(n) * n * n;
    const double norm = 1.0 / (N * N);
    const cplx<T>* f = static_cast<const cplx<T>*>(m.scratch);
    const int lane = int(threadIdx.x) & 63;
    auto twice = [n](int v) { return v != 0 && 2 * v != n ? 2 : 1; };
    auto at = [n](int v, int sign) { return sign != 0 ? n - v : v; };
    for (int pair = int(blockIdx.x) * 4 + (int(threadIdx.x) >> 6); pair < nh * nh;
         pair += int(gridDim.x) * 4) {
        const int a = pair / nh, b = pair - a * nh;
        if (a < b) continue;
        for (int d = lane; d < nh; d += 64) {
            const int bin = int(rint(sqrt(double(a * a + b * b + d * d))));
            if (bin >= nbins) continue;
            // all sixteen loads in flight: an image that is no mode of its own
            // reads its partner again and is left out of the sum
            const int ia = twice(a) - 1, ib = twice(b) - 1, id = twice(d) - 1;
            cplx<T> v[8][2];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int va = at(a, r & ia), vb = at(b, (r >> 1) & ib);
                const cplx<T>* row = f + (int64_t(r < 4 ? va : vb) * n + (r < 4 ? vb : va)) * n;
                v[r][0] = gld(row, d);
                v[r][1] = gld(row, at(d, id));
            }
            double s = 0.0;
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const bool own = (r & 1) <= ia && ((r >> 1) & 1) <= ib && (r < 4 || a != b);
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const cplx<T> w = v[r][k];
                    const double p = double(w.re) * w.re + double(w.im) * w.im;
                    s += own && k <= id ? p : 0.0;
                }
            }
            atomicAdd(&sum[bin], s * norm);
            atomicAdd(&cnt[bin], (unsigned long long)((a != b ? 2 : 1) * twice(a) * twice(b) *
                                                      twice(d)));
        }
    }
    __syncthreads();
    for (int b = int(threadIdx.x); b < nbins; b += 256) {
        gstr(part, int64_t(blockIdx.x) * 2 * nbins + b, sum[b]);
        gstr(part, int64_t(blockIdx.x) * 2 * nbins + nbins + b, double(cnt[b]));
    }
}

// Sixteen of the 2 nbins columns a work-group, sixteen lanes to a column.
__global__ __launch_bounds__(256) void k_shells_finish(const double* __restrict__ part,
                                                       double* __restrict__ out, int nbins,
                                                       int nblocks) {
    __shared__ double red[16][17];
    const int col = int(threadIdx.x) & 15, w = int(threadIdx.x) >> 4;
    const int b = int(blockIdx.x) * 16 + col;
    double s = 0.0;
    if (b < 2 * nbins)
        for (int k = w; k < nblocks; k += 16) s += gldr(part, int64_t(k) * 2 * nbins + b);
    red[w][col] = s;
    __syncthreads();
    if (w != 0 || b >= 2 * nbins) return;
    for (int k = 1; k < 16; ++k) s += red[k][col];
    gstr(out, b, s);
}

hipError_t launch_shells(const Launch& L, int prec, int n, int nbins, double* part, double* out) {
    if (nbins < 1 || nbins > kPkMaxBins) return hipErrorInvalidValue;
    const int g = shell_blocks(n, nbins);
    if (prec)
        k_shells<double><<<g, 256, 0, L.stream>>>(L.members, L.first, nbins, part);
    else
        k_shells<float><<<g, 256, 0, L.stream>>>(L.members, L.first, nbins, part);
    k_shells_finish<<<(2 * nbins + 15) / 16, 256, 0, L.stream>>>(part, out, nbins, g);
    return hipGetLastError();
}

size_t shells_partial_doubles() { return size_t(kPkDoubles) + 2 * kPkMaxBins; }

// FP64 partials of sum |psi - other|^2 and sum |other|^2 (the judge's field
// distance) into part[2 b], part[2 b + 1] over a fixed grid of work-groups,
// then their ordered sums into out[0], out[1].
constexpr int kDistBlocks = 1024;

template <typename T>
__global__ __launch_bounds__(256) void k_distance(const MemberDev* __restrict__ mems, int first,
                                                  const cplx<T>* __restrict__ other, int64_t n,
                                                  double* __restrict__ part) {
    __shared__ double red[2][256];
    const MemberDev& m = mems[first];
    const cplx<T>* psi = static_cast<const cplx<T>*>(m.psi);
    double d = 0.0, o = 0.0;
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n;
         i += int64_t(gridDim.x) * 256) {
        const cplx<T> a = gld(psi, i), b = gld(other, i);
        const double dr = double(a.re) - double(b.re), di = double(a.im) - double(b.im);
        d += dr * dr + di * di;
        o += double(b.re) * double(b.re) + double(b.im) * double(b.im);
    }
    red[0][threadIdx.x] = d;
    red[1][threadIdx.x] = o;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (int(threadIdx.x) < w) {
            red[0][threadIdx.x] += red[0][threadIdx.x + w];
            red[1][threadIdx.x] += red[1][threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        gstr(part, 2 * int64_t(blockIdx.x), red[0][0]);
        gstr(part, 2 * int64_t(blockIdx.x) + 1, red[1][0]);
    }
}

// The two sums of the kDistBlocks partial pairs in a fixed order (thread t
// adds blocks t, t + 256, ..., then the work-group tree).
__global__ __launch_bounds__(256) void k_distance_finish(const double* __restrict__ part,
                                                         double* __restrict__ out) {
    __shared__ double red[2][256];
    const int t = int(threadIdx.x);
    double d = 0.0, o = 0.0;
    for (int b = t; b < kDistBlocks; b += 256) {
        d += gldr(part, 2 * b);
        o += gldr(part, 2 * b + 1);
    }
    red[0][t] = d;
    red[1][t] = o;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w) {
            red[0][t] += red[0][t + w];
            red[1][t] += red[1][t + w];
        }
        __syncthreads();
    }
    if (t != 0) return;
    gstr(out, 0, red[0][0]);
    gstr(out, 1, red[1][0]);
}

hipError_t launch_distance(const Launch& L, int prec, const void* other, int64_t n, double* part,
                           double* out) {
    if (prec)
        k_distance<double><<<kDistBlocks, 256, 0, L.stream>>>(
            L.members, L.first, static_cast<const cplx<double>*>(other), n, part);
    else
        k_distance<float><<<kDistBlocks, 256, 0, L.stream>>>(
            L.members, L.first, static_cast<const cplx<float>*>(other), n, part);
    k_distance_finish<<<1, 256, 0, L.stream>>>(part, out);
    return hipGetLastError();
}

}  // namespace wdm
