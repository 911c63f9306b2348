// Direct spectral sums (Sec. 4.1 eq. DiscreteFT, random-phase reading):
//   Y_c = A sum_j cos(2 pi r_jc),   r_jc = frac-reduced phase in revolutions,
// plus the fused epilogue (K = exp(mu + Y), facies index = #{thresholds below Y}; Secs. 4.1
// and 3.1).  At points: one hardware cosine per mode and point.  On grids the phase splits
// into an x part and a (y,z) part, and the sum is a contraction of their cosines and sines on
// the FP32 matrix cores.
//
// v_cos_f32 / v_sin_f32 take their argument in revolutions; phases are reduced in FP64 first.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "grf_internal.h"

namespace grf {

namespace {

__device__ __forceinline__ float cos_rev(float r) { return __builtin_amdgcn_cosf(r); }

__device__ __forceinline__ void store_out(int64_t c, float yv, const Epi& e, float* __restrict__ y,
                                          float* __restrict__ k, uint8_t* __restrict__ ind)
{
    epi_store(c, yv, e, y, k, ind);
}

// ---------------------------------------------------------------------------- grid, FP32
// The grid sum as a real contraction on the FP32 matrix cores.  Cell centres are symmetric about
// the grid's middle along x: with x = xc + d the mirrored cell has offset -d, and with
// B = a_x d, F = a_x xc + a_y y + a_z z + psi (in revolutions, formed and reduced in FP64)
//   Y(+-d) = E -+ O,   E = sum_j w_j cos F cos B,   O = sum_j w_j sin F sin B,
// so each pair of cells costs two multiply-adds per mode, half of the plain angle sum.  Both
// sums are matrix products (rows the (y, z) pairs, columns the nx / 2 offsets, K the modes) of
// FP32 operands with FP32 accumulation.
//
// A block is eight waves over one tile of TI TS rows x TS columns (2 TS cells along x).  Wave c
// sums the modes of chunk c (an eighth of the table) and makes its operands in registers: lane l
// owns rows l % TS and column l % TS and the mode j + l / TS of each step, two FP64 phases per
// row tile and column and the hardware cosine and sine, the mode's z and phi broadcast from LDS
// (staged 64 modes at a time, private to the wave).  No tables, no barrier in the mode loop.  The
// eight chunk sums meet in LDS and are added in chunk order.  An FP32 matrix step rounds like
// the FMAs of its k values in order (checked bit for bit), so the tile shape changes no result
// bit: a grid and its batched evaluation agree exactly.
//
// What bounds it: 2 flops per mode and cell on the FP32 matrix cores (153 TFLOP/s in a library
// product) plus the operands, about 41 issue cycles per cosine-sine pair: on gfx950 a vector
// instruction does not issue beside another wave's FP32 matrix step (128^3 x 4,096 modes: matrix cores
// busy 60% of the cycles, none of them with vector work), so a 64-row tile's step of 4 x 64 matrix
// cycles costs ~380.  Making four steps' operands together changed nothing.  The plain angle sum on
// the vector units (two FMAs per term on tabulated phases) took, before -> after, one call: 128^3 x
// 4,096 modes 566 -> 175 us, a weighted 517 x 301 x 2,048 table 120 -> 23 us, 64 x 64 x 1,000 27 -> 13 us;
// relative error against FP64 on 128^3 1.6e-6 -> 4.5e-7 (the phases are summed in FP64 and the chunks
// are shorter).
//
// DIRECT_F64 is the same tile on FP64 operands (sincospi of the FP64 fraction) and the FP64 matrix
// cores; its operands, not the products, take the time, so larger grids share each column
// operand among four row tiles.  Tabulated phases and one cospi per mode and cell took, before ->
// after, one call: 64 x 64 x 1,000 modes 22 -> 18 us (what the binding's host work takes),
// 128 x 128 x 2,048 72 -> 20, 300 x 200 x 4,096 420 -> 69, 64^3 x 4,096 1,537 -> 146 us.
constexpr int kDgWaves = 8;    // waves of a block = mode chunks of every sum
constexpr int kDgStage = 64;   // modes staged in LDS per wave
static_assert(kDirectTile == 64, "the batch tile is 64 rows x 32 columns (64 cells)");

__device__ __forceinline__ float sin_rev(float r) { return __builtin_amdgcn_sinf(r); }

typedef float dg_f16 __attribute__((ext_vector_type(16)));
typedef float dg_f4 __attribute__((ext_vector_type(4)));
typedef double dg_d4 __attribute__((ext_vector_type(4)));

template <class R, int TS>
struct DgTile;
template <>
struct DgTile<float, 32> {
    using Acc = dg_f16;
    static __device__ __forceinline__ Acc mma(float a, float b, Acc c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int e, int l) { return 8 * (e >> 2) + 4 * (l >> 5) + (e & 3); }
};
template <>
struct DgTile<float, 16> {
    using Acc = dg_f4;
    static __device__ __forceinline__ Acc mma(float a, float b, Acc c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int e, int l) { return 4 * (l >> 4) + e; }
};
template <>
struct DgTile<double, 16> {
    using Acc = dg_d4;
    static __device__ __forceinline__ Acc mma(double a, double b, Acc c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // (the FP64 form interleaves its output rows across the four lane groups)
    static __device__ __forceinline__ int row(int e, int l) { return 4 * e + (l >> 4); }
};

// Cosine and sine of a phase in revolutions: the hardware's on the fraction in FP32, or FP64.
__device__ __forceinline__ void cos_sin_rev(double t, float& c, float& s)
{
    const float f = static_cast<float>(__builtin_amdgcn_fract(t));
    c = cos_rev(f);
    s = sin_rev(f);
}
__device__ __forceinline__ void cos_sin_rev(double t, double& c, double& s)
{
    sincospi(2.0 * __builtin_amdgcn_fract(t), &s, &c);
}

// Outputs of cell c.
__device__ __forceinline__ void dg_store(const DirectGrid& g, const Epi& epi, int64_t c, float sum)
{
    epi_store(c, g.amp * sum, epi, g.y, g.k, g.ind);
}
__device__ __forceinline__ void dg_store(const DirectGrid& g, const Epi& epi, int64_t c, double sum)
{
    if (g.partial64) {  // one slice of the modes: its raw sums
        g.partial64[static_cast<int64_t>(blockIdx.z) * (g.nq * g.nx) + c] = sum;
        return;
    }
    const double yv = g.amp64 * sum;
    if (g.y64) g.y64[c] = yv;
    if (g.k64) g.k64[c] = exp(g.mu64 + yv);
    if (g.y || g.k || g.ind) epi_store(c, static_cast<float>(yv), epi, g.y, g.k, g.ind);
}

// LDS of one block: the waves' mode stages, later the chunk sums of one row tile.
template <class R, int TS>
struct DgShape {
    static constexpr int kModeB = kDgWaves * kDgStage * (4 * 8 + static_cast<int>(sizeof(R)));
    static constexpr int kSumB = kDgWaves * 2 * TS * TS * static_cast<int>(sizeof(R));
    static constexpr int BYTES = kModeB > kSumB ? kModeB : kSumB;
};

// Rows q0 .. q0 + TI TS - 1, columns i0 .. i0 + TS - 1 (offsets from the middle; column i is cell
// i and its mirror nx - 1 - i).  `smem`: DgShape<R, TS>::BYTES bytes, 16-byte aligned.  Whole block.
template <class R, int TS, int TI, bool WT>
__device__ __forceinline__ void direct_tile(const DirectGrid& g, const Epi& epi, int64_t i0, int64_t q0, char* smem)
{
    using T = DgTile<R, TS>;
    constexpr int KS = 64 / TS;         // modes per matrix step
    constexpr int NE = TS * TS / 64;    // accumulator elements per lane
    constexpr double kInvTwoPi = 0.15915494309189533576888376337251;
    const int t = threadIdx.x, l = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int r = l % TS, kk = l / TS;
    const int nx = g.nx, half = (nx + 1) >> 1;
    const int64_t n = g.n;

    // coordinates times 1 / (2 pi ell): phases in revolutions are plain products with z
    const int64_t ic = min(i0 + r, static_cast<int64_t>(half) - 1);
    const double xc = g.fs[0] * (g.o[0] + 0.5 * static_cast<double>(nx) * g.h[0]);
    const double xd = g.fs[0] * ((static_cast<double>(ic) + 0.5 - 0.5 * static_cast<double>(nx)) * g.h[0]);
    double yy[TI], zz[TI];
#pragma unroll
    for (int i = 0; i < TI; ++i) {
        const int64_t q = min(q0 + i * TS + r, g.nq - 1);
        yy[i] = g.fs[1] * (g.o[1] + (static_cast<double>(q % g.ny) + 0.5) * g.h[1]);
        zz[i] = g.fs[2] * (g.o[2] + (static_cast<double>(q / g.ny) + 0.5) * g.h[2]);
    }

    typename T::Acc ae[TI], ao[TI];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            ae[i][e] = R(0);
            ao[i][e] = R(0);
        }

    // this wave's chunk of the modes (a multiple of 8 modes per chunk, whatever the tile)
    // (FP64: of its slice's modes)
    const int64_t n0 = sizeof(R) == 8 ? static_cast<int64_t>(blockIdx.z) * g.mslice : 0;
    const int64_t n1 = sizeof(R) == 8 ? min(n, n0 + g.mslice) : n;
    const int64_t mc = 8 * ((n1 - n0 + 63) >> 6);
    const int64_t j0 = min(n0 + w * mc, n1), j1 = min(j0 + mc, n1);
    double4* const sm = reinterpret_cast<double4*>(smem) + w * kDgStage;
    R* const sw = reinterpret_cast<R*>(smem + kDgWaves * kDgStage * 32) + w * kDgStage;
    const double* const zx = g.zx;
    const double* const zy = g.zy;
    const double* const z3 = g.zz;

    // modes past the chunk's end stage the table's last entry of the chunk; their row operands
    // are set to zero below
    auto fetch = [&](int64_t j) {
        const int64_t jj = min(j + l, j1 - 1);
        return make_double4(zx[jj], zy[jj], z3 ? z3[jj] : 0.0, g.phi[jj] * kInvTwoPi);
    };
    auto fetch_w = [&](int64_t j) { return WT ? static_cast<R>(g.w[min(j + l, j1 - 1)]) : R(1); };
    double4 nm = make_double4(0.0, 0.0, 0.0, 0.0);
    R nw = R(1);
    if (j0 < j1) {
        nm = fetch(j0);
        nw = fetch_w(j0);
    }
    for (int64_t jb = j0; jb < j1; jb += kDgStage) {
        // the wave's own LDS, read and written in program order: compiler barriers suffice
        __builtin_amdgcn_wave_barrier();
        sm[l] = nm;
        if (WT) sw[l] = nw;
        __builtin_amdgcn_wave_barrier();
        if (jb + kDgStage < j1) {
            nm = fetch(jb + kDgStage);
            nw = fetch_w(jb + kDgStage);
        }
        const int cnt = static_cast<int>(min<int64_t>(kDgStage, j1 - jb));
        auto step = [&](int m, bool tail) {
            const double4 p = sm[m + kk];
            const R wj = WT ? sw[m + kk] : R(1);
            R cb, sb;
            cos_sin_rev(p.x * xd, cb, sb);
            const double base = fma(p.x, xc, p.w);
#pragma unroll
            for (int i = 0; i < TI; ++i) {
                R ca, sa;
                cos_sin_rev(fma(p.z, zz[i], fma(p.y, yy[i], base)), ca, sa);
                if (WT) {
                    ca *= wj;
                    sa *= wj;
                }
                if (tail && m + kk >= cnt) ca = sa = R(0);
                ae[i] = T::mma(ca, cb, ae[i]);
                ao[i] = T::mma(sa, sb, ao[i]);
            }
        };
        int m = 0;
#pragma unroll 4
        for (; m + KS <= cnt; m += KS) step(m, false);
        if (m < cnt) step(m, true);
    }

    // chunk sums -> LDS (element-major: lane-contiguous both ways), added in chunk order
    R* const ss = reinterpret_cast<R*>(smem);
    constexpr int kPart = 2 * TS * TS;  // values per wave: E then O
#pragma unroll
    for (int i = 0; i < TI; ++i) {
        __syncthreads();
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            ss[w * kPart + e * 64 + l] = ae[i][e];
            ss[w * kPart + TS * TS + e * 64 + l] = ao[i][e];
        }
        __syncthreads();
        for (int p = t; p < TS * TS; p += kDgWaves * 64) {
            R se = ss[p], so = ss[TS * TS + p];
#pragma unroll
            for (int c = 1; c < kDgWaves; ++c) {
                se += ss[c * kPart + p];
                so += ss[c * kPart + TS * TS + p];
            }
            const int64_t col = i0 + (p & 63) % TS;
            const int64_t q = q0 + i * TS + T::row(p >> 6, p & 63);
            if (col < half && q < g.nq) {
                const int64_t mirror = nx - 1 - col;
                dg_store(g, epi, q * nx + col, se - so);
                if (mirror != col) dg_store(g, epi, q * nx + mirror, se + so);
            }
        }
    }
}

template <class R, int TS, int TI, bool WT>
__global__ __launch_bounds__(kDgWaves * 64) void k_direct_grid(DirectGrid g, Epi epi, int64_t tiles_i, int64_t tiles)
{
    __shared__ __attribute__((aligned(16))) char smem[DgShape<R, TS>::BYTES];
    const int64_t bid = static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x;
    if (bid >= tiles) return;  // the whole block
    direct_tile<R, TS, TI, WT>(g, epi, bid % tiles_i * TS, bid / tiles_i * (TI * TS), smem);
}

// FP64 sums of the mode slices, added in slice order.
__global__ __launch_bounds__(256) void k_grid_reduce_f64(const double* __restrict__ partial, int slices, int64_t C,
                                                        DirectGrid g, Epi epi)
{
    const int64_t c = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (c >= C) return;
    double v[8];  // at most eight slices: every load in flight
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = partial[static_cast<int64_t>(q < slices ? q : 0) * C + c];
    double sum = v[0];
#pragma unroll
    for (int q = 1; q < 8; ++q)
        if (q < slices) sum += v[q];
    dg_store(g, epi, c, sum);
}

// Persistent batched form: blocks pull (instance, tile) work items from one atomic counter
// until the queue is drained.
__global__ __launch_bounds__(kDgWaves * 64) void k_direct_batch(const DirectBatchItem* __restrict__ items, int n_inst,
                                                               int64_t total, unsigned long long* counter)
{
    __shared__ __attribute__((aligned(16))) char smem[DgShape<float, 32>::BYTES];
    __shared__ unsigned long long s_item;
    for (;;) {
        if (threadIdx.x == 0) s_item = atomicAdd(counter, 1ull);
        __syncthreads();
        const int64_t it = static_cast<int64_t>(s_item);
        __syncthreads();
        if (it >= total) break;
        int lo = 0, hi = n_inst - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (items[mid].item0 <= it) lo = mid;
            else hi = mid - 1;
        }
        const DirectBatchItem& b = items[lo];
        const int64_t local = it - b.item0;
        const int64_t i0 = local % b.tiles_i * 32, q0 = local / b.tiles_i * 64;
        if (b.g.w) direct_tile<float, 32, 2, true>(b.g, b.epi, i0, q0, smem);
        else direct_tile<float, 32, 2, false>(b.g, b.epi, i0, q0, smem);
        __syncthreads();  // the sums in LDS are read before the next item stages over them
    }
}

// ---------------------------------------------------------------------------- points
__device__ __forceinline__ float slice_sum(const float* __restrict__ partial, int slices, int64_t P, int64_t p)
{
    // Sixteen slice loads are in flight at a time; the adds keep slice order.
    constexpr int kGroup = 16;
    float s = 0.f;
    int q = 0;
    for (; q + kGroup <= slices; q += kGroup) {
        float v[kGroup];
#pragma unroll
        for (int u = 0; u < kGroup; ++u) v[u] = partial[static_cast<int64_t>(q + u) * P + p];
#pragma unroll
        for (int u = 0; u < kGroup; ++u) s += v[u];
    }
    for (; q < slices; ++q) s += partial[static_cast<int64_t>(q) * P + p];
    return s;
}

__global__ __launch_bounds__(256) void k_points_reduce(const float* __restrict__ partial, int slices, int64_t P,
                                                      float amp, Epi epi, float* __restrict__ y,
                                                      float* __restrict__ k, uint8_t* __restrict__ ind)
{
    const int64_t p = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p >= P) return;
    store_out(p, amp * slice_sum(partial, slices, P, p), epi, y, k, ind);
}

// Each lane owns R points; every mode's (a_x, a_y, a_z, psi) in revolutions is
// uniform across the block (scalar loads).  The phase a.x + psi is formed and
// reduced in FP64 per mode and point, then the cosine and the sum run in FP32.
// With few points the modes are split over blockIdx.y slices of `mslice` modes each:
// every slice writes its raw partial sums to partial[slice][P] and k_points_reduce adds
// them in slice order and applies the epilogue.
template <int DIM, int R>
__global__ __launch_bounds__(256) void k_direct_points(const double4* __restrict__ prm, const double* __restrict__ wt,
                                                      int n, const double* __restrict__ xyz, int64_t P, float amp,
                                                      Epi epi, float* __restrict__ y, float* __restrict__ k,
                                                      uint8_t* __restrict__ ind, int mslice,
                                                      float* __restrict__ partial)
{
    const int64_t base = static_cast<int64_t>(blockIdx.x) * (256 * R) + threadIdx.x;
    const int j0 = static_cast<int>(blockIdx.y) * mslice;
    const int j1 = min(n, j0 + mslice);
    double px[R], py[R], pz[R];
    float acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t p = min(base + 256 * r, P - 1);
        px[r] = xyz[p * DIM];
        py[r] = xyz[p * DIM + 1];
        pz[r] = DIM == 3 ? xyz[p * DIM + 2] : 0.0;
        acc[r] = 0.f;
    }
    auto mode = [&](const double4& m, float wj) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            double ph = DIM == 3 ? fma(m.z, pz[r], m.w) : m.w;
            ph = fma(m.y, py[r], ph);
            ph = fma(m.x, px[r], ph);
            ph = __builtin_amdgcn_fract(ph);  // x - floor(x) in one FP64 instruction
            acc[r] = fmaf(wj, cos_rev(static_cast<float>(ph)), acc[r]);
        }
    };
    // The (uniform) mode records are loaded four at a time, ahead of their terms; each point
    // still sums the modes in order.
    constexpr int kMG = 4;
    int j = j0;
    for (; j + kMG <= j1; j += kMG) {
        double4 mm[kMG];
        float ww[kMG];
#pragma unroll
        for (int u = 0; u < kMG; ++u) mm[u] = prm[j + u];
        if (wt) {
#pragma unroll
            for (int u = 0; u < kMG; ++u) ww[u] = static_cast<float>(wt[j + u]);
        } else {
#pragma unroll
            for (int u = 0; u < kMG; ++u) ww[u] = 1.f;
        }
#pragma unroll
        for (int u = 0; u < kMG; ++u) mode(mm[u], ww[u]);
    }
    for (; j < j1; ++j) mode(prm[j], wt ? static_cast<float>(wt[j]) : 1.f);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t p = base + 256 * r;
        if (p >= P) continue;
        if (partial) partial[static_cast<int64_t>(blockIdx.y) * P + p] = acc[r];
        else store_out(p, amp * acc[r], epi, y, k, ind);
    }
}

template <int DIM>
__global__ __launch_bounds__(256) void k_direct_points_f64(const double4* __restrict__ prm,
                                                          const double* __restrict__ wt, int n,
                                                          const double* __restrict__ xyz, int64_t P, double amp,
                                                          Epi epi, float* __restrict__ y, float* __restrict__ k,
                                                          uint8_t* __restrict__ ind)
{
    const int64_t p = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p >= P) return;
    const double px = xyz[p * DIM], py = xyz[p * DIM + 1], pz = DIM == 3 ? xyz[p * DIM + 2] : 0.0;
    double s = 0.0;
    for (int j = 0; j < n; ++j) {
        const double4 m = prm[j];
        double ph = fma(m.x, px, fma(m.y, py, fma(m.z, pz, m.w)));
        ph = __builtin_amdgcn_fract(ph);  // x - floor(x) in one FP64 instruction
        s += (wt ? wt[j] : 1.0) * cospi(2.0 * ph);
    }
    store_out(p, static_cast<float>(amp * s), epi, y, k, ind);
}

// ---------------------------------------------------------------------------- epilogue
// Stand-alone epilogue: 4 cells per thread, 16-byte loads and stores.
__global__ __launch_bounds__(256) void k_epilogue(const float* __restrict__ y, int64_t n, Epi epi,
                                                 float* __restrict__ k, uint8_t* __restrict__ ind)
{
    const int64_t n4 = n >> 2;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n4; i += stride) {
        const float4 v = reinterpret_cast<const float4*>(y)[i];
        if (k)
            reinterpret_cast<float4*>(k)[i] =
                make_float4(expf(epi.mu + v.x), expf(epi.mu + v.y), expf(epi.mu + v.z), expf(epi.mu + v.w));
        if (ind) {
            int f0 = 0, f1 = 0, f2 = 0, f3 = 0;
            for (int t = 0; t < epi.nthr; ++t) {
                const float th = epi.thr[t];
                f0 += v.x > th;
                f1 += v.y > th;
                f2 += v.z > th;
                f3 += v.w > th;
            }
            reinterpret_cast<uint32_t*>(ind)[i] = static_cast<uint32_t>(f0) | (static_cast<uint32_t>(f1) << 8) |
                                                  (static_cast<uint32_t>(f2) << 16) | (static_cast<uint32_t>(f3) << 24);
        }
    }
    // ragged tail (n not a multiple of 4)
    if (blockIdx.x == 0 && threadIdx.x < (n & 3)) {
        const int64_t c = n4 * 4 + threadIdx.x;
        store_out(c, y[c], epi, nullptr, k, ind);
    }
}

// Bitruncated rule over two stored fields.
__device__ __forceinline__ int pluri_facies(float a, float b, const PluriEpi& pe)
{
    int i = 0, j = 0;
    for (int q = 0; q < pe.nt; ++q) i += (a > pe.t[q]) ? 1 : 0;
    for (int q = 0; q < pe.ns; ++q) j += (b > pe.s[q]) ? 1 : 0;
    return pe.rule[i * (pe.ns + 1) + j];
}

// Four cells per thread and step (16-byte loads of both fields, one 4-byte facies store and a
// 16-byte value store); the caller guarantees 16-byte aligned fields and value, 4-byte aligned
// facies.  Cells past the last multiple of four go through the per-cell form.
__global__ __launch_bounds__(256) void k_pluri4(const float* __restrict__ y1, const float* __restrict__ y2, int64_t n,
                                               PluriEpi pe, uint8_t* __restrict__ facies, float* __restrict__ value)
{
    const int64_t n4 = n >> 2;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t q = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; q < n4; q += stride) {
        const float4 a = reinterpret_cast<const float4*>(y1)[q];
        const float4 b = reinterpret_cast<const float4*>(y2)[q];
        const int f0 = pluri_facies(a.x, b.x, pe), f1 = pluri_facies(a.y, b.y, pe);
        const int f2 = pluri_facies(a.z, b.z, pe), f3 = pluri_facies(a.w, b.w, pe);
        if (facies)
            reinterpret_cast<uint32_t*>(facies)[q] = static_cast<uint32_t>(f0) | (static_cast<uint32_t>(f1) << 8) |
                                                     (static_cast<uint32_t>(f2) << 16) | (static_cast<uint32_t>(f3) << 24);
        if (value)
            reinterpret_cast<float4*>(value)[q] = make_float4(pe.values[f0], pe.values[f1], pe.values[f2], pe.values[f3]);
    }
    if (blockIdx.x == 0 && threadIdx.x < (n & 3)) {
        const int64_t c = n4 * 4 + threadIdx.x;
        const int f = pluri_facies(y1[c], y2[c], pe);
        if (facies) facies[c] = static_cast<uint8_t>(f);
        if (value) value[c] = pe.values[f];
    }
}

// The rule straight from both fields' slice sums (the order and rounding of k_points_reduce), the
// fields stored only where the caller keeps them: one pass over the sums in place of three launches.
// Bound by its launch and one pass over the sums: 5.7 us at 1024 x 512 cells against 4.75 + 4.75 +
// 4.35 us for the three, the whole call 64 -> 58 us.
__global__ __launch_bounds__(256) void k_pluri_slices(const float* __restrict__ p1, const float* __restrict__ p2,
                                                     int slices, int64_t n, float amp1, float amp2, PluriEpi pe,
                                                     uint8_t* __restrict__ facies, float* __restrict__ value,
                                                     float* __restrict__ y1, float* __restrict__ y2)
{
    const int64_t c = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (c >= n) return;
    const float a = amp1 * slice_sum(p1, slices, n, c), b = amp2 * slice_sum(p2, slices, n, c);
    const int f = pluri_facies(a, b, pe);
    if (y1) y1[c] = a;
    if (y2) y2[c] = b;
    if (facies) facies[c] = static_cast<uint8_t>(f);
    if (value) value[c] = pe.values[f];
}

// One cell per thread and step (unaligned buffers).
__global__ __launch_bounds__(256) void k_pluri(const float* __restrict__ y1, const float* __restrict__ y2, int64_t n,
                                              PluriEpi pe, uint8_t* __restrict__ facies, float* __restrict__ value)
{
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t c = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; c < n; c += stride) {
        const int f = pluri_facies(y1[c], y2[c], pe);
        if (facies) facies[c] = static_cast<uint8_t>(f);
        if (value) value[c] = pe.values[f];
    }
}

__global__ __launch_bounds__(256) void k_epilogue_scalar(const float* __restrict__ y, int64_t n, Epi epi,
                                                        float* __restrict__ k, uint8_t* __restrict__ ind)
{
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t c = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; c < n; c += stride)
        store_out(c, y[c], epi, nullptr, k, ind);
}

}  // namespace

namespace {
template <class R, int TS, int TI>
hipError_t launch_direct_tile(const DirectGrid& g, const Epi& epi, hipStream_t s, int slices = 1)
{
    const int64_t half = (static_cast<int64_t>(g.nx) + 1) / 2;
    const int64_t ti = (half + TS - 1) / TS, tq = (g.nq + TI * TS - 1) / (TI * TS);
    const int64_t tiles = ti * tq;
    // more threads along x than 32 bits count are silently dropped: more tiles fold into y
    const int64_t gy = (tiles + kMaxGridX - 1) / kMaxGridX;
    if (gy > 65535) return hipErrorInvalidValue;
    const dim3 grid(static_cast<unsigned>((tiles + gy - 1) / gy), static_cast<unsigned>(gy), static_cast<unsigned>(slices));
    if (g.w)
        hipLaunchKernelGGL((k_direct_grid<R, TS, TI, true>), grid, dim3(kDgWaves * 64), 0, s, g, epi, ti, tiles);
    else
        hipLaunchKernelGGL((k_direct_grid<R, TS, TI, false>), grid, dim3(kDgWaves * 64), 0, s, g, epi, ti, tiles);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_direct_grid_f32(const DirectGrid& g, const Epi& epi, hipStream_t s)
{
    const int64_t half = (static_cast<int64_t>(g.nx) + 1) / 2;
    auto tiles = [&](int64_t rows, int64_t cols) { return ((half + cols - 1) / cols) * ((g.nq + rows - 1) / rows); };
    // A tile's time does not depend on how many there are until the CUs are full, and grows with
    // its area: the widest tile that fills most of the 256 CUs.  Kernel time in us with 256 / 1,024 /
    // 4,096 modes for 64 x 32, 32 x 32 and 16 x 16: 64^3 (64 tiles of 64 x 32) 11 / 27 / 91, 7.6 / 17 / 52
    // and 7.0 / 15 / 41; 1024 x 512 (128) 12 / 28 / 95, 8.2 / 18 / 56 and 10 / 23 / 74; 100 x 90 x 80 (226)
    // 12 / 29 / 99, 12 / 31 / 104 and 17 / 41 / 142; 128^3 (512) 20 / 54 / 191, 21 / 58 / 204 and 28 / 80 /
    // 273.
    if (tiles(64, 32) >= 160) return launch_direct_tile<float, 32, 2>(g, epi, s);
    if (tiles(32, 32) >= 192) return launch_direct_tile<float, 32, 1>(g, epi, s);
    return launch_direct_tile<float, 16, 1>(g, epi, s);
}

hipError_t launch_direct_grid_f64(const DirectGrid& g0, const Epi& epi, double* ws, size_t ws_doubles, hipStream_t s)
{
    DirectGrid g = g0;
    g.mslice = g.n;
    g.partial64 = nullptr;
    const int64_t half = (static_cast<int64_t>(g.nx) + 1) / 2, C = g.nq * g.nx;
    // An operand costs several matrix steps: four row tiles per column operand once they fill most CUs.
    // Kernel time in us, four / one, with 256 and 1,000 modes: 512 x 512 (128 tiles of 64 rows) 19 / 14
    // and 52 / 38; 700 x 600 (220) 21 / 24 and 53 / 70; 1024 x 512 (256) 21 / 25 and 54 / 72.  (Five
    // operands for 64 rows, two for 16: one is the better up to 32 rows: 65,536 x 1 cells x 1,000
    // modes 121 us for 361.)
    if (g.nq > 32 && ((half + 15) / 16) * ((g.nq + 63) / 64) >= 192)
        return launch_direct_tile<double, 16, 4>(g, epi, s);
    // Few tiles: slices of at least 128 modes spread the operands over more CUs (a second launch adds
    // the slices in order, about 3 us), where the workspace holds their sums.  64 x 64 (8 tiles),
    // whole / in slices: 256 modes 7.8 / 8.6 us, 1,000 19 / 9.6, 4,096 63 / 16; 128 x 128 (32) 7.8 / 8.9,
    // 19 / 11, 64 / 24.
    const int64_t tiles = ((half + 15) / 16) * ((g.nq + 15) / 16);
    int64_t sl = std::min<int64_t>(std::min<int64_t>(128 / tiles, 8), g.n / 128);
    if (g.n < 384) sl = 1;
    sl = std::min<int64_t>(sl, static_cast<int64_t>(ws_doubles) / C);
    if (sl < 2) return launch_direct_tile<double, 16, 1>(g, epi, s);
    g.mslice = (g.n + sl - 1) / sl;
    g.partial64 = ws;
    const int slices = static_cast<int>((g.n + g.mslice - 1) / g.mslice);
    const hipError_t e = launch_direct_tile<double, 16, 1>(g, epi, s, slices);
    if (e != hipSuccess) return e;
    g.partial64 = nullptr;
    hipLaunchKernelGGL(k_grid_reduce_f64, dim3(static_cast<unsigned>((C + 255) / 256)), dim3(256), 0, s, ws, slices, C,
                       g, epi);
    return hipGetLastError();
}

hipError_t launch_direct_points(const double* params, const double* w, int64_t n, int dim, const double* xyz,
                                int64_t P, bool fp64, float amp, const Epi& epi, float* y, float* k, uint8_t* ind,
                                float* partial, hipStream_t s)
{
    const double4* prm = reinterpret_cast<const double4*>(params);
    if (fp64) {
        const int64_t blocks = (P + 255) / 256;
        if (blocks > 0x7fffffff) return hipErrorInvalidValue;
        if (dim == 3)
            hipLaunchKernelGGL(k_direct_points_f64<3>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, prm, w,
                               static_cast<int>(n), xyz, P, static_cast<double>(amp), epi, y, k, ind);
        else
            hipLaunchKernelGGL(k_direct_points_f64<2>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, prm, w,
                               static_cast<int>(n), xyz, P, static_cast<double>(amp), epi, y, k, ind);
        return hipGetLastError();
    }
    constexpr int R = kPointsPerLane;
    const int64_t blocks = (P + 256 * R - 1) / (256 * R);
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    const int slices = points_mode_slices(P, n);
    const int mslice = static_cast<int>((n + slices - 1) / slices);
    float* part = slices > 1 ? partial : nullptr;
    const dim3 g(static_cast<unsigned>(blocks), static_cast<unsigned>(slices));
    if (dim == 3)
        hipLaunchKernelGGL((k_direct_points<3, R>), g, dim3(256), 0, s, prm, w, static_cast<int>(n), xyz, P, amp, epi,
                           y, k, ind, mslice, part);
    else
        hipLaunchKernelGGL((k_direct_points<2, R>), g, dim3(256), 0, s, prm, w, static_cast<int>(n), xyz, P, amp, epi,
                           y, k, ind, mslice, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || slices == 1) return e;
    hipLaunchKernelGGL(k_points_reduce, dim3(static_cast<unsigned>((P + 255) / 256)), dim3(256), 0, s, partial, slices,
                       P, amp, epi, y, k, ind);
    return hipGetLastError();
}

hipError_t launch_points_reduce(const float* partial, int slices, int64_t P, float amp, const Epi& epi, float* y,
                                float* k, uint8_t* ind, hipStream_t s)
{
    hipLaunchKernelGGL(k_points_reduce, dim3(static_cast<unsigned>((P + 255) / 256)), dim3(256), 0, s, partial, slices,
                       P, amp, epi, y, k, ind);
    return hipGetLastError();
}

int bin_mode_slices(int64_t P, int64_t n)
{
    // about 8192 work-item waves (several per SIMD); each slice keeps >= 64 modes
    if (P <= 0 || n <= 0) return 1;
    const int64_t waves = (P + kBinItemSlots - 1) / kBinItemSlots;
    int64_t s = (8192 + waves - 1) / waves;
    s = std::min<int64_t>(s, std::max<int64_t>(n / 64, 1));
    s = std::min<int64_t>(s, 64);
    return static_cast<int>(std::max<int64_t>(s, 1));
}

int points_mode_slices(int64_t P, int64_t n)
{
    // Enough blocks to fill 256 CUs several times over; each slice keeps >= 64 modes.
    if (P <= 0 || n <= 0) return 1;
    const int64_t pblocks = (P + 256 * kPointsPerLane - 1) / (256 * kPointsPerLane);
    int64_t s = (2048 + pblocks - 1) / pblocks;
    s = std::min<int64_t>(s, std::max<int64_t>(n / 64, 1));
    s = std::min<int64_t>(s, 64);
    return static_cast<int>(std::max<int64_t>(s, 1));
}

hipError_t launch_direct_batch(const DirectBatchItem* items, int n_inst, int64_t total, unsigned long long* counter,
                               int grid, hipStream_t s)
{
    hipLaunchKernelGGL(k_direct_batch, dim3(grid), dim3(kDgWaves * 64), 0, s, items, n_inst, total, counter);
    return hipGetLastError();
}

int direct_batch_blocks_per_cu()
{
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_direct_batch, kDgWaves * 64, 0) != hipSuccess) return 1;
    return nb > 0 ? nb : 1;
}

hipError_t launch_pluri_slices(const float* p1, const float* p2, int slices, int64_t n, float amp1, float amp2,
                               const PluriEpi& pe, uint8_t* facies, float* value, float* y1, float* y2, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pluri_slices, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, s, p1, p2, slices, n,
                       amp1, amp2, pe, facies, value, y1, y2);
    return hipGetLastError();
}

hipError_t launch_pluri_epilogue(const float* y1, const float* y2, int64_t n, const PluriEpi& pe, uint8_t* facies,
                                 float* value, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const bool aligned = reinterpret_cast<uintptr_t>(y1) % 16 == 0 && reinterpret_cast<uintptr_t>(y2) % 16 == 0 &&
                         reinterpret_cast<uintptr_t>(value) % 16 == 0 && reinterpret_cast<uintptr_t>(facies) % 4 == 0;
    if (aligned) {
        int64_t blocks = ((n >> 2) + 255) / 256;
        if (blocks < 1) blocks = 1;
        if (blocks > 256 * 64) blocks = 256 * 64;
        hipLaunchKernelGGL(k_pluri4, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, y1, y2, n, pe, facies,
                           value);
        return hipGetLastError();
    }
    int64_t blocks = (n + 255) / 256;
    if (blocks > 256 * 64) blocks = 256 * 64;
    hipLaunchKernelGGL(k_pluri, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, y1, y2, n, pe, facies, value);
    return hipGetLastError();
}

hipError_t launch_epilogue(const float* y, int64_t n, const Epi& epi, float* k, uint8_t* ind, hipStream_t s)
{
    const bool aligned = (reinterpret_cast<uintptr_t>(y) % 16 == 0) && (reinterpret_cast<uintptr_t>(k) % 16 == 0) &&
                         (reinterpret_cast<uintptr_t>(ind) % 4 == 0);
    if (!aligned) {
        int64_t blocks = (n + 255) / 256;
        if (blocks > 256 * 64) blocks = 256 * 64;
        hipLaunchKernelGGL(k_epilogue_scalar, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, y, n, epi, k, ind);
        return hipGetLastError();
    }
    const int64_t n4 = n >> 2;
    int64_t blocks = (n4 + 255) / 256;
    if (blocks < 1) blocks = 1;
    if (blocks > 256 * 64) blocks = 256 * 64;
    hipLaunchKernelGGL(k_epilogue, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, y, n, epi, k, ind);
    return hipGetLastError();
}

}  // namespace grf
