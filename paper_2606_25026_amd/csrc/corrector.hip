// Learned coarse-grid corrector: a three-layer 3x3x3 convolution network
// (3 -> C -> C -> 2 channels, circular padding, ReLU after the hidden layers)
// with BF16 weights and activations on MFMA and FP32 accumulation, its
// backward pass (data and weight gradients, split-K FP32 partials with a
// fixed-order reduction) and Adam.  The network is not part of the paper's
// method; it corrects a 2x-coarser split-step run toward the fine one.
//
// Convolution as an implicit GEMM: out[cell][m] = sum_k W[m][k] in[cell + tap(k)][c(k)]
// with k = tap * CP + c (CP = channels padded to 4 or 16).  One wavefront owns
// 16 cells along z and all 16 (padded) output channels, and issues one
// v_mfma_f32_16x16x16_bf16 per K-chunk of 16:
//   A (16 x 16, M x K): lane l holds W[l % 16][chunk*16 + 4*(l/16) + q], q < 4
//   B (16 x 16, K x N): lane l holds in[cell(l % 16) + tap][c + q] for
//                       k = chunk*16 + 4*(l/16) + q
//   D (16 x 16, M x N): lane l holds out[cell(l % 16)][4*(l/16) + q]
#include "wdm_internal.hpp"

#include <cstdint>

namespace wdm {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// float -> bf16, round to nearest even (NaN kept quiet)
__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) != 0x7f800000u) u += 0x7fffu + ((u >> 16) & 1u);
    return uint16_t(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float(uint32_t(h) << 16); }

// Epilogue modes of the convolution kernel.
enum ConvEpi : int {
    kEpiBiasReluBf16 = 0,   // out = bf16(relu(acc + bias)), CPOUT channels
    kEpiBiasF32 = 1,        // out = f32(acc + bias), COUT channels (network output)
    kEpiMaskBf16 = 2,       // out = bf16(acc * (mask > 0)), CPOUT channels (backward data)
    // the correction (COUT = 2): out is psi (f32 re, im per cell),
    // psi += s_out (acc + bias) with s_out = scal[5], and part[work-group] gets
    // the FP64 sum of the corrected |psi|^2 over the work-group's cells
    kEpiApply = 3,
};

// Convolution tile: 4 x 4 x 16 output cells (x, y, z) per work-group pass.
// The input brick with its one-cell periodic halo, 6 x 6 x 18 cells, is staged
// in LDS once and read by all 27 taps; each wavefront owns the four 16-cell z
// segments of one x row (N = 16 cells per MFMA) and keeps its A operand (the
// layer's weights, all K chunks) in registers for the whole launch.
constexpr int kCTX = 4, kCTY = 4, kCTZ = 16;
constexpr int kCBX = kCTX + 2, kCBY = kCTY + 2, kCBZ = kCTZ + 2;
constexpr int kCBrick = kCBX * kCBY * kCBZ;

// The input brick of tile t: every 8-byte word of its cells (one 16-byte half
// cell per thread and slot for 16 channels, one 8-byte cell for 4), loaded into
// registers; stored to LDS by brick_store.
template <int W8>
struct BrickRegs {
    static constexpr int kWords = kCBrick * W8;              // 8-byte words
    static constexpr int kPer = W8 == 4 ? 2 : 1;             // words per load
    static constexpr int kLoads = kWords / kPer;
    static constexpr int kIt = (kLoads + 255) / 256;
    u32x4 v[W8 == 4 ? kIt : 1];
    uint64_t w[W8 == 4 ? 1 : kIt];
};

// Tile t's first cell.
struct ConvTile {
    int x0, y0, z0;
    __device__ __forceinline__ ConvTile(int t, int ty, int tz) {
        const int r = t / tz, q = r / ty;
        x0 = q * kCTX;
        y0 = (r - q * ty) * kCTY;
        z0 = (t - r * tz) * kCTZ;
    }
};

// The brick cell of each of this lane's loads, one byte a coordinate: the same in
// every tile, so a load's address is six additions and compares (with the cell
// and its three wraps found by division each time the address work of a tile was
// more than its MFMAs': 16 -> 16 channels at 128^3 64 and 71 us, now 57 and 64).
template <int W8>
struct BrickCells {
    using B = BrickRegs<W8>;
    int cell[B::kIt];
    __device__ __forceinline__ BrickCells() {
#pragma unroll
        for (int k = 0; k < B::kIt; ++k) {
            const int c = (int(threadIdx.x) + k * 256) / (W8 / B::kPer);
            const int rr = c / kCBZ, bx = rr / kCBY;
            cell[k] = bx << 16 | (rr - bx * kCBY) << 8 | (c - rr * kCBZ);
        }
    }
};

// v in [-1, n + kCTZ]: the periodic index, inside the grid; beyond the first node
// past the end any (no valid output reads it).
__device__ __forceinline__ int wrap_edge(int v, int n) {
    return v < 0 ? v + n : min(v >= n ? v - n : v, n - 1);
}

template <int CPIN, int W8>
__device__ __forceinline__ void brick_load(BrickRegs<W8>& R, const BrickCells<W8>& C,
                                           const uint16_t* __restrict__ in, const ConvTile& t,
                                           int n) {
    using B = BrickRegs<W8>;
    const int tid = int(threadIdx.x);
#pragma unroll
    for (int k = 0; k < B::kIt; ++k) {
        const int i = tid + k * 256;
        if (i < B::kLoads) {
            const int c = C.cell[k];
            // (a cell's channels end below 2^32 bytes: n <= 512)
            const uint32_t g = uint32_t((wrap_edge(t.x0 + (c >> 16) - 1, n) * n +
                                         wrap_edge(t.y0 + (c >> 8 & 255) - 1, n)) * n +
                                        wrap_edge(t.z0 + (c & 255) - 1, n));
            if constexpr (W8 == 4)
                R.v[k] = *(const WDM_GAS u32x4*)(in + uint64_t(g) * CPIN + (i & 1) * 8);
            else
                R.w[k] = *(const WDM_GAS uint64_t*)(in + uint64_t(g) * CPIN);
        }
    }
}

template <int W8>
__device__ __forceinline__ void brick_store(const BrickRegs<W8>& R, uint64_t* brick) {
    using B = BrickRegs<W8>;
    const int tid = int(threadIdx.x);
#pragma unroll
    for (int k = 0; k < B::kIt; ++k) {
        const int i = tid + k * 256;
        if (i < B::kLoads) {
            if constexpr (W8 == 4)
                reinterpret_cast<u32x4*>(brick)[i] = R.v[k];
            else
                brick[i] = R.w[k];
        }
    }
}

// in: bf16 [cells][CPIN]; wmat: bf16 [16][KC*16] (rows >= COUT zero);
// out: see ConvEpi.  COUT real output channels (<= 16), CPOUT padded store width.
// Persistent: work-group b handles tiles b, b + gridDim.x, ...; the next
// tile's brick is loaded into registers while the current one is computed.
// The layer's weights (the MFMA A operand) sit in LDS, rows padded by four
// entries so the sixteen rows a wavefront reads fall on different banks.
// Two output channels (FEW) would leave 14 of the MFMA's 16 rows empty: its rows
// are then the channels of the three dy taps, a brick row is multiplied once for
// all of them, and the three partial sums of an output meet by two lane swaps:
// 54 products of a wavefront's tile instead of 108, 54 -> 43 us at 128^3.
template <int CPIN, int COUT, int CPOUT, int EPI>
__global__ __launch_bounds__(256, 3) void k_conv(const uint16_t* __restrict__ in,
                                                 const uint16_t* __restrict__ wmat,
                                                 const float* __restrict__ bias,
                                                 const uint16_t* __restrict__ mask, void* out,
                                                 int n, const double* __restrict__ scal,
                                                 double* __restrict__ part) {
    constexpr int KC = (27 * CPIN + 15) / 16;
    constexpr int KW = KC * 16 + 4;              // LDS row of the weights (bf16 entries)
    constexpr int W8 = CPIN / 4;                 // 8-byte words per brick cell
    __shared__ __align__(16) uint64_t brick[kCBrick * W8];
    __shared__ __align__(16) uint16_t wl[16 * KW];
    const int tid = int(threadIdx.x);
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int col = lane & 15;                   // z within the segment; A row
    const int kq = lane >> 4;                    // which 4-wide k group
    for (int i = tid; i < 16 * KC * 4; i += 256) {
        const int row = i / (KC * 4), q = i - row * (KC * 4);
        *reinterpret_cast<uint64_t*>(&wl[row * KW + 4 * q]) =
            *(const WDM_GAS uint64_t*)(wmat + int64_t(row) * (KC * 16) + 4 * q);
    }
    auto a_op = [&](int ch) {
        bf16x4 a;
        const uint64_t w = *reinterpret_cast<const uint64_t*>(&wl[col * KW + ch * 16 + 4 * kq]);
        __builtin_memcpy(&a, &w, sizeof(a));
        return a;
    };
    const int tx = (n + kCTX - 1) / kCTX, ty = (n + kCTY - 1) / kCTY, tz = (n + kCTZ - 1) / kCTZ;
    const int ntiles = tx * ty * tz;
    const BrickCells<W8> cells;
    BrickRegs<W8> R;
    if (int(blockIdx.x) < ntiles)
        brick_load<CPIN, W8>(R, cells, in, ConvTile(int(blockIdx.x), ty, tz), n);
    double mass = 0.0;   // kEpiApply: this lane's cells, in tile order
    const float s_out = EPI == kEpiApply ? float(gldr(scal, 5)) : 0.0f;
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const ConvTile tile(t, ty, tz);
        const int x0 = tile.x0, y0 = tile.y0, z0 = tile.z0;
        brick_store<W8>(R, brick);
        __syncthreads();
        const int next = t + int(gridDim.x);
        if (next < ntiles) brick_load<CPIN, W8>(R, cells, in, ConvTile(next, ty, tz), n);
        // wavefront `wave` owns x = x0 + wave, y = y0 + s (s < 4), z = z0 + col
        constexpr bool FEW = COUT == 2 && CPIN == 16;
        constexpr int NACC = FEW ? kCTY + 2 : kCTY;
        f32x4 acc[NACC];
#pragma unroll
        for (int s2 = 0; s2 < NACC; ++s2) acc[s2] = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (FEW) {
            // row 4 dy + o of A: channel o (rows 2 and 3 of the weights are zero)
            // of tap (dx, dy, dz); acc[rr]: brick row rr, lane group dy
            const int dy = min(col >> 2, 2);
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                for (int dz = 0; dz < 3; ++dz) {
                    uint64_t w = *reinterpret_cast<const uint64_t*>(
                        &wl[(col & 3) * KW + (dx * 9 + dy * 3 + dz) * 16 + 4 * kq]);
                    if (col >= 12) w = 0;
                    bf16x4 a;
                    __builtin_memcpy(&a, &w, sizeof(a));
#pragma unroll
                    for (int rr = 0; rr < kCTY + 2; ++rr) {
                        const uint64_t bw =
                            brick[(((wave + dx) * kCBY + rr) * kCBZ + col + dz) * W8 + kq];
                        bf16x4 b;
                        __builtin_memcpy(&b, &bw, sizeof(b));
                        acc[rr] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc[rr], 0, 0, 0);
                    }
                }
        } else if constexpr (CPIN == 16) {
            // one K chunk per tap (16 channels).  For fixed (dx, dz) the four
            // segments and three dy offsets read only six brick rows (segment
            // s at offset dy is row s + dy): each B operand read from LDS
            // serves two MFMAs on average.
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                for (int dz = 0; dz < 3; ++dz) {
                    uint64_t braw[kCTY + 2];
#pragma unroll
                    for (int rr = 0; rr < kCTY + 2; ++rr)
                        braw[rr] = brick[(((wave + dx) * kCBY + rr) * kCBZ + col + dz) * W8 + kq];
#pragma unroll
                    for (int dy = 0; dy < 3; ++dy) {
                        const bf16x4 a = a_op(dx * 9 + dy * 3 + dz);
#pragma unroll
                        for (int s2 = 0; s2 < kCTY; ++s2) {
                            bf16x4 b;
                            __builtin_memcpy(&b, &braw[s2 + dy], sizeof(b));
                            acc[s2] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc[s2], 0,
                                                                                0, 0);
                        }
                    }
                }
        } else {
#pragma unroll
            for (int ch = 0; ch < KC; ++ch) {
                const int k0 = ch * 16 + 4 * kq;
                const int tap = k0 / CPIN, c = k0 % CPIN;
                const bool live = k0 < 27 * CPIN;
                const int dx = tap / 9, dy = (tap / 3) % 3, dz = tap % 3;
                const int cell0 = ((wave + dx) * kCBY + dy) * kCBZ + col + dz;
                const bf16x4 a = a_op(ch);
#pragma unroll
                for (int s2 = 0; s2 < kCTY; ++s2) {
                    const uint64_t bw = live ? brick[(cell0 + s2 * kCBZ) * W8 + c / 4] : 0ull;
                    bf16x4 b;
                    __builtin_memcpy(&b, &bw, sizeof(b));
                    acc[s2] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc[s2], 0, 0, 0);
                }
            }
        }
        // epilogue: lane holds out[cell][4*kq + q] of each segment
        const int x = x0 + wave, z = z0 + col, m0 = 4 * kq;
        if constexpr (FEW) {
            // lane group dy holds brick row s + dy's share of output row s; the
            // sum lands in every group, and group s keeps row s
            float o2[2] = {0.0f, 0.0f};
#pragma unroll
            for (int s2 = 0; s2 < kCTY; ++s2)
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    float v = kq == 0   ? acc[s2][o]
                              : kq == 1 ? acc[s2 + 1][o]
                              : kq == 2 ? acc[s2 + 2][o]
                                        : 0.0f;
                    v += __shfl_xor(v, 16);
                    v += __shfl_xor(v, 32);
                    if (kq == s2) o2[o] = v;
                }
            const int y = y0 + kq;
            if (x < n && y < n && z < n) {
                const int64_t cell = (int64_t(x) * n + y) * n + z;
                float* to = static_cast<float*>(out);   // (the correction: psi)
                float re = o2[0] + gldr(bias, 0), im = o2[1] + gldr(bias, 1);
                if constexpr (EPI == kEpiApply) {
                    re = gldr(to, 2 * cell) + s_out * re;
                    im = gldr(to, 2 * cell + 1) + s_out * im;
                    mass += double(re) * double(re) + double(im) * double(im);
                }
                gstr(to, 2 * cell, re);
                gstr(to, 2 * cell + 1, im);
            }
        } else {
            static_assert(EPI == kEpiBiasReluBf16 || EPI == kEpiMaskBf16, "bf16 outputs");
#pragma unroll
            for (int s2 = 0; s2 < kCTY; ++s2) {
                const int y = y0 + s2;
                if (x >= n || y >= n || z >= n || m0 >= CPOUT) continue;
                const int64_t cell = (int64_t(x) * n + y) * n + z;
                uint16_t rq[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float v = acc[s2][q];
                    if constexpr (EPI == kEpiBiasReluBf16) {
                        v = m0 + q < COUT ? fmaxf(v + gldr(bias, m0 + q), 0.0f) : 0.0f;
                    } else {
                        const float mk = bf2f(gldr(mask, cell * CPOUT + m0 + q));
                        v = (m0 + q < COUT && mk > 0.0f) ? v : 0.0f;
                    }
                    rq[q] = f2bf(v);
                }
                const uint64_t packed = uint64_t(rq[0]) | (uint64_t(rq[1]) << 16) |
                                        (uint64_t(rq[2]) << 32) | (uint64_t(rq[3]) << 48);
                gstr(reinterpret_cast<uint64_t*>(static_cast<uint16_t*>(out)),
                     (cell * CPOUT + m0) / 4, packed);
            }
        }
        __syncthreads();   // the next tile's brick overwrites this one
    }
    if constexpr (EPI == kEpiApply) {
        // the work-group's sum in a fixed order (lanes, then the four
        // wavefronts), reusing the brick's LDS
        double* red = reinterpret_cast<double*>(brick);
        red[tid] = mass;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if (tid < w) red[tid] += red[tid + w];
            __syncthreads();
        }
        if (tid == 0) gstr(part, int64_t(blockIdx.x), red[0]);
    }
}

// ---------------------------------------------------------------------------
// Weight gradients.  gw[m][c][tap] = sum_p dz[p][m] act[p + tap][c] is a GEMM
// whose K dimension is the cells; both operands are stored channels last, so
// the K index runs across memory.  What bounded the direct form (each lane
// gathering its operand two bytes at a time from global memory, neighbour
// indices by 64-bit division) was the load instructions: 1.65 / 5.92 / 5.93 ms
// for the three layers at 128^3.  Here a work-group stages a brick of both
// operands in LDS transposed to [channel][x][y][z] once per tile and every tap
// reads it from there: a lane's eight K values are eight neighbouring z of one
// channel, one 16-byte LDS read for v_mfma_f32_16x16x32_bf16.
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// 4 x 4 x 32 cells per tile; bricks with the one-cell periodic halo.
constexpr int kGX = 4, kGY = 4, kGZ = 32;
constexpr int kGBX = kGX + 2, kGBY = kGY + 2, kGRows = kGBX * kGBY;
constexpr int kGWaves = 8, kGThreads = 64 * kGWaves;
// bytes of one z row in LDS (32 cells, two halo cells, padding) and of one
// channel: odd multiples of 16 bytes, so that sixteen channels read at once
// fall on different banks
constexpr int kGRow = 80;
constexpr int kGChanIn = kGRows * kGRow + 16;        // haloed brick
constexpr int kGChanOut = kGX * kGY * kGRow + 16;    // the tile's own cells

__device__ __forceinline__ bf16x8 lds_b128(const uint8_t* p) {
    const u32x4 w = *reinterpret_cast<const u32x4*>(p);
    bf16x8 r;
    __builtin_memcpy(&r, &w, sizeof(r));
    return r;
}
__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 w) {
    bf16x8 r;
    __builtin_memcpy(&r, &w, sizeof(r));
    return r;
}
// (a, b) hold 8 channels of the cells z and z + 1; word k of the result pairs
// channel k of both: (z | z + 1 << 16)
__device__ __forceinline__ uint32_t pair_channel(u32x4 a, u32x4 b, int k) {
    const uint32_t x = a[k >> 1], y = b[k >> 1];
    return (k & 1) ? __builtin_amdgcn_perm(y, x, 0x07060302u) : __builtin_amdgcn_perm(y, x, 0x05040100u);
}

struct GTile {
    int x0, y0, z0;
    __device__ __forceinline__ GTile(int64_t t, int ty, int tz) {
        const int64_t r = t / tz;
        z0 = int(t - r * tz) * kGZ;
        const int64_t q = r / ty;
        y0 = int(r - q * ty) * kGY;
        x0 = int(q) * kGX;
    }
};

// 16-channel operand without halo: item i = ((row * 16) + pair) * 2 + half,
// one item per thread; cells past the grid give zeros.
static_assert(kGX * kGY * (kGZ / 2) * 2 == kGThreads, "one item per thread");
struct OutRegs {
    u32x4 a, b;
    __device__ __forceinline__ void load(const uint16_t* __restrict__ src, const GTile& t, int n) {
        const int i = int(threadIdx.x), half = i & 1, pair = (i >> 1) & 15, row = i >> 5;
        const int x = t.x0 + row / kGY, y = t.y0 + row % kGY, z = t.z0 + 2 * pair;
        a = b = u32x4{0u, 0u, 0u, 0u};
        if (x < n && y < n) {
            const uint16_t* p = src + ((int64_t(x) * n + y) * n + z) * 16 + half * 8;
            if (z < n) a = *(const WDM_GAS u32x4*)p;
            if (z + 1 < n) b = *(const WDM_GAS u32x4*)(p + 16);
        }
    }
    __device__ __forceinline__ void store(uint8_t* lds) const {
        const int i = int(threadIdx.x), half = i & 1, pair = (i >> 1) & 15, row = i >> 5;
        uint8_t* p = lds + half * 8 * kGChanOut + row * kGRow + pair * 4;
#pragma unroll
        for (int k = 0; k < 8; ++k)
            *reinterpret_cast<uint32_t*>(p + k * kGChanOut) = pair_channel(a, b, k);
    }
};

// 16-channel operand with halo: items ((row * 17) + pair) * 2 + half of the
// 6 x 6 x 34 brick.  Only halo cells wrap; cells beyond them are zeros.
struct HaloRegs {
    static constexpr int kPairs = kGZ / 2 + 1, kItems = kGRows * kPairs * 2;
    static constexpr int kIt = (kItems + kGThreads - 1) / kGThreads;
    u32x4 a[kIt], b[kIt];
    __device__ __forceinline__ void load(const uint16_t* __restrict__ src, const GTile& t, int n) {
#pragma unroll
        for (int k = 0; k < kIt; ++k) {
            const int i = int(threadIdx.x) + k * kGThreads;
            a[k] = b[k] = u32x4{0u, 0u, 0u, 0u};
            if (i >= kItems) continue;
            const int half = i & 1, j = i >> 1, row = j / kPairs, pair = j - row * kPairs;
            const int x = t.x0 + row / kGBY - 1, y = t.y0 + row % kGBY - 1, z = t.z0 + 2 * pair - 1;
            if (x > n || y > n) continue;
            const uint16_t* p =
                src + (int64_t(wrap_edge(x, n)) * n + wrap_edge(y, n)) * n * 16 + half * 8;
            if (z <= n) a[k] = *(const WDM_GAS u32x4*)(p + int64_t(wrap_edge(z, n)) * 16);
            if (z < n) b[k] = *(const WDM_GAS u32x4*)(p + int64_t(wrap_edge(z + 1, n)) * 16);
        }
    }
    __device__ __forceinline__ void store(uint8_t* lds) const {
#pragma unroll
        for (int k = 0; k < kIt; ++k) {
            const int i = int(threadIdx.x) + k * kGThreads;
            if (i >= kItems) continue;
            const int half = i & 1, j = i >> 1, row = j / kPairs, pair = j - row * kPairs;
            uint8_t* p = lds + half * 8 * kGChanIn + row * kGRow + pair * 4;
#pragma unroll
            for (int c = 0; c < 8; ++c)
                *reinterpret_cast<uint32_t*>(p + c * kGChanIn) = pair_channel(a[k], b[k], c);
        }
    }
};

// 4-channel operand with halo, kept as three copies shifted by 0, 1 and 2
// cells along z, so that every tap's read is 16-byte aligned: copy s holds
// cell z0 - 1 + i + s at position i.
struct Halo4Regs {
    static constexpr int kPairs = kGZ / 2 + 1, kItems = kGRows * kPairs;
    static constexpr int kIt = (kItems + kGThreads - 1) / kGThreads;
    uint64_t p0[kIt], p1[kIt], p2[kIt];
    __device__ __forceinline__ void load(const uint16_t* __restrict__ src, const GTile& t, int n) {
#pragma unroll
        for (int k = 0; k < kIt; ++k) {
            const int i = int(threadIdx.x) + k * kGThreads;
            p0[k] = p1[k] = p2[k] = 0ull;
            if (i >= kItems) continue;
            const int row = i / kPairs, pair = i - row * kPairs;
            const int x = t.x0 + row / kGBY - 1, y = t.y0 + row % kGBY - 1, z = t.z0 + 2 * pair - 1;
            if (x > n || y > n) continue;
            const uint16_t* p = src + (int64_t(wrap_edge(x, n)) * n + wrap_edge(y, n)) * n * 4;
            if (z <= n) p0[k] = *(const WDM_GAS uint64_t*)(p + int64_t(wrap_edge(z, n)) * 4);
            if (z < n) p1[k] = *(const WDM_GAS uint64_t*)(p + int64_t(wrap_edge(z + 1, n)) * 4);
            if (z + 1 < n && pair + 1 < kPairs)
                p2[k] = *(const WDM_GAS uint64_t*)(p + int64_t(wrap_edge(z + 2, n)) * 4);
        }
    }
    __device__ __forceinline__ void store(uint8_t* lds) const {
#pragma unroll
        for (int k = 0; k < kIt; ++k) {
            const int i = int(threadIdx.x) + k * kGThreads;
            if (i >= kItems) continue;
            const int row = i / kPairs, pair = i - row * kPairs;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t v0 = uint32_t(p0[k] >> (16 * c)) & 0xffffu,
                               v1 = uint32_t(p1[k] >> (16 * c)) & 0xffffu,
                               v2 = uint32_t(p2[k] >> (16 * c)) & 0xffffu;
                uint8_t* p = lds + c * kGChanIn + row * kGRow + pair * 4;
                if (pair + 1 < kPairs) {
                    *reinterpret_cast<uint32_t*>(p) = v0 | (v1 << 16);
                    *reinterpret_cast<uint32_t*>(p + 4 * kGChanIn) = v1 | (v2 << 16);
                }
                if (pair > 0) *reinterpret_cast<uint32_t*>(p + 8 * kGChanIn - 4) = v0 | (v1 << 16);
            }
        }
    }
};

// Sum of the wavefronts' accumulators (NT 16 x 16 tiles each) in a fixed
// order, written as part[tile][row][col].
template <int NT>
__device__ __forceinline__ void wgrad_write(float* lds, const f32x4* acc, float* dst) {
    const int tid = int(threadIdx.x), lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, kq = lane >> 4;
    __syncthreads();   // the bricks are no longer read
#pragma unroll
    for (int round = 0; round < 2; ++round) {
        if (wave / 4 == round) {
            float* b = lds + (wave & 3) * (NT * 256);
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float* e = b + t * 256 + (4 * kq + q) * 16 + col;
                    *e = round ? *e + acc[t][q] : acc[t][q];
                }
        }
        __syncthreads();
    }
    for (int i = tid; i < NT * 256; i += kGThreads)
        gstr(dst, i, (lds[i] + lds[i + NT * 256]) + (lds[i + 2 * NT * 256] + lds[i + 3 * NT * 256]));
}

constexpr int kGTiles16 = 28;   // 27 taps and the bias (columns all equal)
constexpr int kGTiles4 = 8;     // 7 groups of four taps and the bias

// Hidden layer: 16 x 16 channels.  M = dz channel, N = act channel, one
// accumulator tile per tap (112 registers a wavefront).  A lane reads ten
// cells of an act row once and forms the three z taps from them; each
// wavefront takes two of the tile's sixteen (x, y) rows.  Register prefetch of
// the next tile, one LDS copy, one work-group of eight wavefronts per CU (the
// partials' capacity).
__global__ __launch_bounds__(kGThreads) void k_wgrad16(const uint16_t* __restrict__ dz,
                                                       const uint16_t* __restrict__ act,
                                                       float* __restrict__ part, int n) {
    constexpr int kBrick = 16 * kGChanIn + 16 * kGChanOut;
    constexpr int kSum = 4 * kGTiles16 * 256 * 4;
    __shared__ __align__(16) uint8_t lds[kBrick > kSum ? kBrick : kSum];
    uint8_t* la = lds;                     // act
    uint8_t* lz = lds + 16 * kGChanIn;     // dz
    const int lane = int(threadIdx.x) & 63, wave = int(threadIdx.x) >> 6;
    const int ch = lane & 15, kq = lane >> 4;
    const int tx = (n + kGX - 1) / kGX, ty = (n + kGY - 1) / kGY, tz = (n + kGZ - 1) / kGZ;
    const int64_t ntiles = int64_t(tx) * ty * tz;
    const bf16x8 ones = as_bf16x8(u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
    f32x4 acc[kGTiles16];
#pragma unroll
    for (int t = 0; t < kGTiles16; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    HaloRegs ra;
    OutRegs rz;
    int64_t t = blockIdx.x;
    if (t < ntiles) {
        const GTile g(t, ty, tz);
        ra.load(act, g, n);
        rz.load(dz, g, n);
    }
    for (; t < ntiles; t += gridDim.x) {
        const GTile g0(t, ty, tz);
        ra.store(la);
        rz.store(lz);
        __syncthreads();
        if (t + gridDim.x < ntiles) {
            const GTile g(t + gridDim.x, ty, tz);
            ra.load(act, g, n);
            rz.load(dz, g, n);
        }
#pragma unroll 1
        for (int rr = 0; rr < 2; ++rr) {
            const int row = wave * 2 + rr, rx = row / kGY, ry = row % kGY;
            if (g0.x0 + rx >= n || g0.y0 + ry >= n) continue;   // uniform over the wavefront
            const bf16x8 a = lds_b128(lz + ch * kGChanOut + row * kGRow + kq * 16);
            acc[27] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, ones, acc[27], 0, 0, 0);
#pragma unroll
            for (int d = 0; d < 9; ++d) {
                const uint8_t* p =
                    la + ch * kGChanIn + ((rx + d / 3) * kGBY + ry + d % 3) * kGRow + kq * 16;
                const u32x4 w = *reinterpret_cast<const u32x4*>(p);
                const uint32_t e = *reinterpret_cast<const uint32_t*>(p + 16);
                const u32x4 w1 = {__builtin_amdgcn_alignbit(w[1], w[0], 16),
                                  __builtin_amdgcn_alignbit(w[2], w[1], 16),
                                  __builtin_amdgcn_alignbit(w[3], w[2], 16),
                                  __builtin_amdgcn_alignbit(e, w[3], 16)};
                const u32x4 w2 = {w[1], w[2], w[3], e};
                acc[3 * d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, as_bf16x8(w), acc[3 * d], 0, 0, 0);
                acc[3 * d + 1] =
                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, as_bf16x8(w1), acc[3 * d + 1], 0, 0, 0);
                acc[3 * d + 2] =
                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, as_bf16x8(w2), acc[3 * d + 2], 0, 0, 0);
            }
        }
        __syncthreads();   // the next tile's bricks overwrite these
    }
    wgrad_write<kGTiles16>(reinterpret_cast<float*>(lds), acc,
                           part + int64_t(blockIdx.x) * (kGTiles16 * 256));
}

// The layers with a 4-channel side: `big` (16 channels) at the tile's cells,
// `small` (4 channels) at the cell plus the tap.  M = big channel, N = (tap of
// a group of four, small channel): 7 MFMAs per 32 cells where one per tap
// would leave twelve of sixteen rows or columns empty.
//   first layer: big = dz, small = act, the bias sums big;
//   last layer: big = act, small = dz at p' = p - tap, so tap group entries are
//   the mirrored taps; the bias sums the centre tap's small (BIAS_SMALL), its
//   rows masked to the grid.
template <bool BIAS_SMALL>
__global__ __launch_bounds__(kGThreads) void k_wgrad4(const uint16_t* __restrict__ big,
                                                      const uint16_t* __restrict__ small,
                                                      float* __restrict__ part, int n) {
    constexpr int kBrick = 12 * kGChanIn + 16 * kGChanOut;
    constexpr int kSum = 4 * kGTiles4 * 256 * 4;
    __shared__ __align__(16) uint8_t lds[kBrick > kSum ? kBrick : kSum];
    uint8_t* ls = lds;                     // small, three shifted copies
    uint8_t* lb = lds + 12 * kGChanIn;     // big
    const int lane = int(threadIdx.x) & 63, wave = int(threadIdx.x) >> 6;
    const int ch = lane & 15, kq = lane >> 4;
    const int tx = (n + kGX - 1) / kGX, ty = (n + kGY - 1) / kGY, tz = (n + kGZ - 1) / kGZ;
    const int64_t ntiles = int64_t(tx) * ty * tz;
    // this lane's tap and channel of each group: LDS offset of its row
    int off[7];
#pragma unroll
    for (int g = 0; g < 7; ++g) {
        const int tap = min(4 * g + (ch >> 2), 26);   // the 28th entry is not used
        off[g] = ((tap % 3) * 4 + (ch & 3)) * kGChanIn + ((tap / 9) * kGBY + (tap / 3) % 3) * kGRow +
                 kq * 16;
    }
    f32x4 acc[kGTiles4];
#pragma unroll
    for (int t = 0; t < kGTiles4; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    Halo4Regs rs;
    OutRegs rb;
    int64_t t = blockIdx.x;
    if (t < ntiles) {
        const GTile g(t, ty, tz);
        rs.load(small, g, n);
        rb.load(big, g, n);
    }
    for (; t < ntiles; t += gridDim.x) {
        const GTile g0(t, ty, tz);
        rs.store(ls);
        rb.store(lb);
        __syncthreads();
        if (t + gridDim.x < ntiles) {
            const GTile g(t + gridDim.x, ty, tz);
            rs.load(small, g, n);
            rb.load(big, g, n);
        }
        // ones at the cells inside the grid along z
        u32x4 ow;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int z = g0.z0 + 8 * kq + 2 * k;
            ow[k] = (z < n ? 0x3f80u : 0u) | (z + 1 < n ? 0x3f800000u : 0u);
        }
        const bf16x8 ones = as_bf16x8(ow);
#pragma unroll 1
        for (int rr = 0; rr < 2; ++rr) {
            const int row = wave * 2 + rr, rx = row / kGY, ry = row % kGY;
            if (g0.x0 + rx >= n || g0.y0 + ry >= n) continue;   // uniform over the wavefront
            const bf16x8 a = lds_b128(lb + ch * kGChanOut + row * kGRow + kq * 16);
            const uint8_t* p = ls + (rx * kGBY + ry) * kGRow;
#pragma unroll
            for (int g = 0; g < 7; ++g) {
                const bf16x8 b = lds_b128(p + off[g]);
                acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[g], 0, 0, 0);
                if (BIAS_SMALL && g == 3)   // the centre tap is entry 1 of group 3
                    acc[7] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, b, acc[7], 0, 0, 0);
            }
            if (!BIAS_SMALL) acc[7] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, ones, acc[7], 0, 0, 0);
        }
        __syncthreads();
    }
    wgrad_write<kGTiles4>(reinterpret_cast<float*>(lds), acc,
                          part + int64_t(blockIdx.x) * (kGTiles4 * 256));
}

// Fixed-order sum of the work-groups' partials, straight into the parameter
// layout w[co][ci][27], b[co].  64 entries per work-group, each by four lanes
// over a quarter of the partials (one lane over all of them was 20 us a layer,
// a chain of 256 dependent loads' latency).
template <int LAYER>
__global__ __launch_bounds__(256) void k_wgrad_sum(const float* __restrict__ part, int nblocks,
                                                   float* __restrict__ gw, float* __restrict__ gb) {
    constexpr int NT = LAYER == 1 ? kGTiles16 : kGTiles4;
    constexpr int LEN = NT * 256;
    __shared__ float red[4][64];
    const int e = int(threadIdx.x) & 63, seg = int(threadIdx.x) >> 6;
    const int i = int(blockIdx.x) * 64 + e;
    const int per = (nblocks + 3) / 4, b0 = seg * per, b1 = min(nblocks, b0 + per);
    float s = 0.0f;
    int b = b0;
    for (; b + 16 <= b1; b += 16) {
        float v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = gldr(part, int64_t(b + k) * LEN + i);
#pragma unroll
        for (int k = 0; k < 16; ++k) s += v[k];
    }
    for (; b < b1; ++b) s += gldr(part, int64_t(b) * LEN + i);
    red[seg][e] = s;
    __syncthreads();
    if (seg != 0) return;
    s = (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]);
    const int tile = i >> 8, row = (i >> 4) & 15, col = i & 15;
    if constexpr (LAYER == 1) {
        if (tile < 27)
            gstr(gw, (int64_t(row) * 16 + col) * 27 + tile, s);
        else if (col == 0)
            gstr(gb, row, s);
    } else {
        const int entry = 4 * tile + (col >> 2), c = col & 3;
        if (tile < 7) {
            if (LAYER == 0 && entry < 27 && c < 3) gstr(gw, (int64_t(row) * 3 + c) * 27 + entry, s);
            if (LAYER == 2 && entry < 27 && c < 2)
                gstr(gw, (int64_t(c) * 16 + row) * 27 + (26 - entry), s);
        } else {
            if (LAYER == 0 && col == 0) gstr(gb, row, s);
            if (LAYER == 2 && row == 0 && (col >> 2) == 1 && c < 2) gstr(gb, c, s);
        }
    }
}

// ---- packing, loss, Adam ---------------------------------------------------

// f32 [cells][CIN] -> bf16 [cells][4] (zero padded), a cell a lane (a value a lane,
// its indices by 64-bit division: 23 us at 128^3, now 12); channels scaled by sc[0]
// and, from the third on, sc[1] (the network's input scales, device doubles) when
// sc is given.
template <int CIN>
__global__ __launch_bounds__(256) void k_pack_bf16(const float* __restrict__ x,
                                                   uint64_t* __restrict__ y, int64_t cells,
                                                   const double* __restrict__ sc) {
    const int64_t p = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (p >= cells) return;
    uint64_t w = 0;
#pragma unroll
    for (int c = 0; c < CIN; ++c) {
        float v = gldr(x, p * CIN + c);
        if (sc) v *= float(gldr(sc, c < 2 ? 0 : 1));
        w |= uint64_t(f2bf(v)) << (16 * c);
    }
    gstr(y, p, w);
}

// loss = sum (y - t)^2 / count in FP64 partials over two channels; dy = bf16(2 (y -
// t) / count), stored with four.  A cell a lane (28 us at 128^3 as above, now 12).
// The target t is in the network's output units divided by s_out (read
// from *s_out when given): the network learns t / s_out.
__global__ __launch_bounds__(256) void k_mse(const float* __restrict__ y, const float* __restrict__ t,
                                             uint64_t* __restrict__ dy, double* __restrict__ part,
                                             int64_t cells, const double* __restrict__ s_out) {
    __shared__ double red[256];
    const int64_t count = cells * 2;
    const float inv = s_out ? float(1.0 / gldr(s_out, 0)) : 1.0f;
    double s = 0.0;
    for (int64_t p = int64_t(blockIdx.x) * 256 + threadIdx.x; p < cells;
         p += int64_t(gridDim.x) * 256) {
        uint64_t w = 0;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const float d = gldr(y, p * 2 + c) - gldr(t, p * 2 + c) * inv;
            s += double(d) * double(d);
            w |= uint64_t(f2bf(float(2.0 * double(d) / double(count)))) << (16 * c);
        }
        gstr(dy, p, w);
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (int(threadIdx.x) < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) gstr(part, int64_t(blockIdx.x), red[0] / double(count));
}

// Adam on FP32 master parameters (bias-corrected step count t).
__global__ void k_adam(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ mo,
                       float* __restrict__ ve, int n, float lr, float b1, float b2, float eps,
                       float c1, float c2) {
    const int i = int(blockIdx.x) * 256 + int(threadIdx.x);
    if (i >= n) return;
    const float gi = gldr(g, i);
    const float m = b1 * gldr(mo, i) + (1.0f - b1) * gi;
    const float v = b2 * gldr(ve, i) + (1.0f - b2) * gi * gi;
    gstr(mo, i, m);
    gstr(ve, i, v);
    gstr(w, i, gldr(w, i) - lr * (m / c1) / (sqrtf(v / c2) + eps));
}

// Lay out FP32 weights w[co][ci][27] as the MFMA A matrices:
//   fwd[m][k]  = w[m][c][tap]            k = tap * CPIN + c
//   bwd[m][k]  = w[co][m][26 - tap]      k = tap * CPOUT + co   (transposed, flipped)
__global__ void k_pack_weights(const float* __restrict__ w, uint16_t* __restrict__ fwd,
                               uint16_t* __restrict__ bwd, int cin, int cout, int cpin, int cpout) {
    const int kcf = (27 * cpin + 15) / 16 * 16;
    const int kcb = (27 * cpout + 15) / 16 * 16;
    const int i = int(blockIdx.x) * 256 + int(threadIdx.x);
    if (i < 16 * kcf) {
        const int m = i / kcf, k = i % kcf;
        const int tap = k / cpin, c = k % cpin;
        float v = 0.0f;
        if (m < cout && k < 27 * cpin && c < cin) v = gldr(w, (int64_t(m) * cin + c) * 27 + tap);
        gstr(fwd, i, f2bf(v));
    }
    if (bwd && i < 16 * kcb) {
        const int m = i / kcb, k = i % kcb;
        const int tap = k / cpout, co = k % cpout;
        float v = 0.0f;
        if (m < cin && k < 27 * cpout && co < cout)
            v = gldr(w, (int64_t(co) * cin + m) * 27 + (26 - tap));
        gstr(bwd, i, f2bf(v));
    }
}

// ---- the corrector applied to a member's state -------------------------------
// scal (device doubles): [1] mass before, [2] mass after, [3] s_psi, [4] s_phi,
// [5] s_out.  Reductions: a fixed grid of kMassBlocks work-groups, each
// summing a fixed range into its own FP64 partial (deterministic).
constexpr int kMassBlocks = 1024;

__device__ __forceinline__ double block_sum(double v, double* red) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (int(threadIdx.x) < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    return red[0];
}

// Network inputs from the state, x0[p] = bf16(Re psi s_psi, Im psi s_psi,
// Phi s_phi, 0), and the FP64 partials of |psi|^2 (mass before the correction).
__global__ __launch_bounds__(256) void k_state_pack(const float* __restrict__ psi,
                                                    const float* __restrict__ phi,
                                                    uint16_t* __restrict__ x0, int64_t cells,
                                                    const double* __restrict__ scal,
                                                    double* __restrict__ part) {
    __shared__ double red[256];
    const float sp = float(gldr(scal, 3)), sf = float(gldr(scal, 4));
    double m = 0.0;
    for (int64_t p = int64_t(blockIdx.x) * 256 + threadIdx.x; p < cells;
         p += int64_t(gridDim.x) * 256) {
        const float re = gldr(psi, 2 * p), im = gldr(psi, 2 * p + 1);
        m += double(re) * double(re) + double(im) * double(im);
        const uint64_t packed = uint64_t(f2bf(re * sp)) | (uint64_t(f2bf(im * sp)) << 16) |
                                (uint64_t(f2bf(gldr(phi, p) * sf)) << 32);
        gstr(reinterpret_cast<uint64_t*>(x0), p, packed);
    }
    const double t = block_sum(m, red);
    if (threadIdx.x == 0) gstr(part, int64_t(blockIdx.x), t);
}

// out[slot] = sum of n partials in a fixed order (thread t adds t, t + 256,
// ..., then the work-group tree), one 256-thread work-group.
__global__ __launch_bounds__(256) void k_sum_parts(const double* __restrict__ part, int n,
                                                   double* __restrict__ out, int slot) {
    __shared__ double red[256];
    double s = 0.0;
    for (int i = int(threadIdx.x); i < n; i += 256) s += gldr(part, i);
    const double t = block_sum(s, red);
    if (threadIdx.x == 0) gstr(out, slot, t);
}

// psi *= sqrt(mass before / mass after), the factor formed in FP64.
__global__ void k_rescale(float* __restrict__ psi, int64_t cells, const double* __restrict__ scal) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i >= 2 * cells) return;
    const double a = gldr(scal, 2);
    const float f = a > 0.0 ? float(sqrt(gldr(scal, 1) / a)) : 1.0f;
    gstr(psi, i, gldr(psi, i) * f);
}

// ---- training data --------------------------------------------------------
// A training pair from a member's state and a target field: x[p] = (Re psi,
// Im psi, Phi), y[p] = (Re, Im)(target - psi), both f32 channels last.
__global__ void k_pair(const float* __restrict__ psi, const float* __restrict__ phi,
                       const float* __restrict__ target, float* __restrict__ x,
                       float* __restrict__ y, int64_t cells) {
    const int64_t p = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (p >= cells) return;
    const float re = gldr(psi, 2 * p), im = gldr(psi, 2 * p + 1);
    gstr(x, 3 * p + 0, re);
    gstr(x, 3 * p + 1, im);
    gstr(x, 3 * p + 2, gldr(phi, p));
    gstr(y, 2 * p + 0, gldr(target, 2 * p) - re);
    gstr(y, 2 * p + 1, gldr(target, 2 * p + 1) - im);
}

// Moments of a training set, accumulated pair by pair into per-work-group
// FP64 rows (first pair: overwrite): [0] sum x0^2 + x1^2, [1] sum x2,
// [2] sum x2^2, [3] sum y0^2 + y1^2, [4] sum y0 + y1.
constexpr int kMoments = 5;
__global__ __launch_bounds__(256) void k_moments(const float* __restrict__ x,
                                                 const float* __restrict__ y, int64_t cells,
                                                 double* __restrict__ rows, int first) {
    __shared__ double red[256];
    double a[kMoments] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int64_t p = int64_t(blockIdx.x) * 256 + threadIdx.x; p < cells;
         p += int64_t(gridDim.x) * 256) {
        const double x0 = gldr(x, 3 * p), x1 = gldr(x, 3 * p + 1), x2 = gldr(x, 3 * p + 2);
        const double y0 = gldr(y, 2 * p), y1 = gldr(y, 2 * p + 1);
        a[0] += x0 * x0 + x1 * x1;
        a[1] += x2;
        a[2] += x2 * x2;
        a[3] += y0 * y0 + y1 * y1;
        a[4] += y0 + y1;
    }
    for (int f = 0; f < kMoments; ++f) {
        const double t = block_sum(a[f], red);
        if (threadIdx.x == 0) {
            double* r = rows + int64_t(blockIdx.x) * kMoments + f;
            gstr(r, 0, first ? t : gldr(r, 0) + t);
        }
        __syncthreads();
    }
}

// Scales from the moments of `count` cells (count = pairs x cells per pair):
// s_psi = 1 / rms|psi|, s_phi = 1 / std(Phi), s_out = std of the residual's
// components (population moments); written to scal[3..5].
__global__ __launch_bounds__(256) void k_fit_scales(const double* __restrict__ rows, double count,
                                                    double* __restrict__ scal) {
    __shared__ double red[256];
    double m[kMoments];
    for (int f = 0; f < kMoments; ++f) {
        double s = 0.0;
        for (int b = int(threadIdx.x); b < kMassBlocks; b += 256)
            s += gldr(rows, int64_t(b) * kMoments + f);
        m[f] = block_sum(s, red);
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    const double ms = m[0] / count;
    const double mean_phi = m[1] / count, var_phi = m[2] / count - mean_phi * mean_phi;
    const double mean_y = m[4] / (2.0 * count), var_y = m[3] / (2.0 * count) - mean_y * mean_y;
    gstr(scal, 3, ms > 0.0 ? 1.0 / sqrt(ms) : 1.0);
    gstr(scal, 4, var_phi > 0.0 ? 1.0 / sqrt(var_phi) : 1.0);
    gstr(scal, 5, var_y > 0.0 ? sqrt(var_y) : 1e-30);
}

__global__ void k_set_scales(double* __restrict__ scal, double s_psi, double s_phi, double s_out) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    gstr(scal, 3, s_psi);
    gstr(scal, 4, s_phi);
    gstr(scal, 5, s_out);
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
// Persistent grid of the convolution: one work-group per tile up to `per_cu`
// per compute unit.  Eight at 4 input channels; three at 16, what their 146 to 150
// VGPRs hold (34.7 KB of LDS would hold four): at 128^3 the forward pass takes 129 us
// and its 16 -> 16 layer 57, 66 with four launched per CU, the fourth of which waits
// until another ends.
static unsigned conv_blocks(int n, int per_cu) {
    static int cus = 0;
    if (cus == 0) {
        int dev = 0, c = 0;
        cus = (hipGetDevice(&dev) == hipSuccess &&
               hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
               c > 0) ? c : 256;
    }
    const int64_t tiles = int64_t((n + kCTX - 1) / kCTX) * ((n + kCTY - 1) / kCTY) *
                          ((n + kCTZ - 1) / kCTZ);
    const int64_t cap = int64_t(per_cu) * cus;
    return unsigned(tiles < cap ? tiles : cap);
}

hipError_t conv_forward_layer(hipStream_t s, int layer, const uint16_t* in, const uint16_t* w,
                              const float* b, void* out, int n) {
    if (layer == 0)
        k_conv<4, 16, 16, kEpiBiasReluBf16><<<conv_blocks(n, 8), 256, 0, s>>>(in, w, b, nullptr,
                                                                             out, n, nullptr, nullptr);
    else if (layer == 1)
        k_conv<16, 16, 16, kEpiBiasReluBf16><<<conv_blocks(n, 3), 256, 0, s>>>(in, w, b, nullptr,
                                                                              out, n, nullptr, nullptr);
    else
        k_conv<16, 2, 4, kEpiBiasF32><<<conv_blocks(n, 3), 256, 0, s>>>(in, w, b, nullptr, out, n,
                                                                        nullptr, nullptr);
    return hipGetLastError();
}

// Gradient wrt the input of layer `layer` (1 or 2), masked by that input's ReLU.
hipError_t conv_backward_data(hipStream_t s, int layer, const uint16_t* dz, const uint16_t* wbwd,
                              const uint16_t* act_in, uint16_t* dact, int n) {
    if (layer == 2)
        k_conv<4, 16, 16, kEpiMaskBf16><<<conv_blocks(n, 8), 256, 0, s>>>(dz, wbwd, nullptr,
                                                                         act_in, dact, n,
                                                                         nullptr, nullptr);
    else
        k_conv<16, 16, 16, kEpiMaskBf16><<<conv_blocks(n, 3), 256, 0, s>>>(dz, wbwd, nullptr,
                                                                          act_in, dact, n,
                                                                          nullptr, nullptr);
    return hipGetLastError();
}

// Floats of one work-group's weight-gradient partials, at most.
int wgrad_part_floats() { return kGTiles16 * 256; }

// Gradients of layer `layer`'s weights and biases into gw, gb: partials of at
// most `max_blocks` work-groups in `part`, then their fixed-order sum.
hipError_t conv_backward_weight(hipStream_t s, int layer, const uint16_t* dz,
                                const uint16_t* act_in, float* part, int max_blocks, float* gw,
                                float* gb, int n) {
    const int64_t tiles = int64_t((n + kGX - 1) / kGX) * ((n + kGY - 1) / kGY) *
                          ((n + kGZ - 1) / kGZ);
    // one work-group per CU (LDS of the 16-channel kernel), two of the others;
    // their partials are under a third of its
    const int nb = int(tiles < max_blocks ? tiles : max_blocks);
    const int nb2 = int(tiles < 2 * max_blocks ? tiles : 2 * max_blocks);
    if (layer == 1) {
        k_wgrad16<<<nb, kGThreads, 0, s>>>(dz, act_in, part, n);
        k_wgrad_sum<1><<<kGTiles16 * 4, 256, 0, s>>>(part, nb, gw, gb);
    } else if (layer == 0) {
        k_wgrad4<false><<<nb2, kGThreads, 0, s>>>(dz, act_in, part, n);
        k_wgrad_sum<0><<<kGTiles4 * 4, 256, 0, s>>>(part, nb2, gw, gb);
    } else {
        k_wgrad4<true><<<nb2, kGThreads, 0, s>>>(act_in, dz, part, n);
        k_wgrad_sum<2><<<kGTiles4 * 4, 256, 0, s>>>(part, nb2, gw, gb);
    }
    return hipGetLastError();
}

hipError_t net_pack_input(hipStream_t s, const float* x, uint16_t* y, int64_t cells, int cin,
                          const double* scales) {
    const unsigned g = unsigned((cells + 255) / 256);
    uint64_t* out = reinterpret_cast<uint64_t*>(y);
    if (cin == 3)
        k_pack_bf16<3><<<g, 256, 0, s>>>(x, out, cells, scales);
    else if (cin == 2)
        k_pack_bf16<2><<<g, 256, 0, s>>>(x, out, cells, scales);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t net_mse(hipStream_t s, const float* y, const float* t, uint16_t* dy, double* part,
                   double* out, int64_t cells, const double* s_out) {
    constexpr int kBlocks = 1024;
    k_mse<<<kBlocks, 256, 0, s>>>(y, t, reinterpret_cast<uint64_t*>(dy), part, cells, s_out);
    k_sum_parts<<<1, 256, 0, s>>>(part, kBlocks, out, 0);
    return hipGetLastError();
}

hipError_t net_adam(hipStream_t s, float* w, const float* g, float* m, float* v, int n, float lr,
                    float b1, float b2, float eps, float c1, float c2) {
    k_adam<<<(n + 255) / 256, 256, 0, s>>>(w, g, m, v, n, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t net_pack_weights(hipStream_t s, const float* w, uint16_t* fwd, uint16_t* bwd, int cin,
                            int cout, int cpin, int cpout) {
    const int len = 16 * ((27 * (cpin > cpout ? cpin : cpout) + 15) / 16 * 16);
    k_pack_weights<<<(len + 255) / 256, 256, 0, s>>>(w, fwd, bwd, cin, cout, cpin, cpout);
    return hipGetLastError();
}

hipError_t net_state_pack(hipStream_t s, const float* psi, const float* phi, uint16_t* x0,
                          int64_t cells, double* scal, double* part) {
    k_state_pack<<<kMassBlocks, 256, 0, s>>>(psi, phi, x0, cells, scal, part);
    k_sum_parts<<<1, 256, 0, s>>>(part, kMassBlocks, scal, 1);
    return hipGetLastError();
}

// The network's last layer with the correction in its epilogue: psi +=
// s_out (layer output), the corrected mass summed per work-group and then in
// a fixed order into scal[2]; with `rescale`, psi *= sqrt(scal[1] / scal[2]).
hipError_t net_last_layer_apply(hipStream_t s, const uint16_t* in, const uint16_t* w,
                                const float* b, float* psi, int n, double* scal, double* part,
                                bool rescale) {
    const unsigned g = conv_blocks(n, 3);
    if (g > unsigned(kMassBlocks)) return hipErrorInvalidValue;   // the partials' capacity
    k_conv<16, 2, 4, kEpiApply><<<g, 256, 0, s>>>(in, w, b, nullptr, psi, n, scal, part);
    k_sum_parts<<<1, 256, 0, s>>>(part, int(g), scal, 2);
    const int64_t cells = int64_t(n) * n * n;
    if (rescale) k_rescale<<<unsigned((2 * cells + 255) / 256), 256, 0, s>>>(psi, cells, scal);
    return hipGetLastError();
}


hipError_t net_pair(hipStream_t s, const float* psi, const float* phi, const float* target,
                    float* x, float* y, int64_t cells) {
    k_pair<<<unsigned((cells + 255) / 256), 256, 0, s>>>(psi, phi, target, x, y, cells);
    return hipGetLastError();
}

hipError_t net_moments(hipStream_t s, const float* x, const float* y, int64_t cells, double* rows,
                       bool first) {
    k_moments<<<kMassBlocks, 256, 0, s>>>(x, y, cells, rows, first ? 1 : 0);
    return hipGetLastError();
}

hipError_t net_fit_scales(hipStream_t s, const double* rows, double count, double* scal) {
    k_fit_scales<<<1, 256, 0, s>>>(rows, count, scal);
    return hipGetLastError();
}

hipError_t net_set_scales(hipStream_t s, double* scal, double s_psi, double s_phi, double s_out) {
    k_set_scales<<<1, 64, 0, s>>>(scal, s_psi, s_phi, s_out);
    return hipGetLastError();
}

size_t net_moment_doubles() { return size_t(kMassBlocks) * kMoments; }

}  // namespace wdm
