// Split-precision grid sum folded over the grid's middle (the hi+lo separable forms).
//
// Cell centres are symmetric about the middle along x: with x = xc + d the mirrored cell has
// offset -d, and with B = a_x d and F = a_x xc + a_y y + a_z z + psi (Sec. 4.1 phases),
//   Y(+-d) = E -+ O,   E = sum_j w_j cos F cos B,   O = sum_j w_j sin F sin B,
// so each pair of cells costs two real multiply-adds per mode, half of the complex product
// P_z Q of the separable form.  E and O are matrix products on the 16-bit matrix cores (rows
// the (y, z) pairs, columns the nx / 2 offsets, K the modes), every factor split hi + lo and
// the three products hi hi, hi lo, lo hi accumulated in FP32.
//
// Operands: per-axis tables (phases formed and reduced in FP64), eight modes of one axis point in
// 64 contiguous bytes, [ldp / 8][points][64 B].  The columns (and the rows of a 2-D grid) are
// stored split, [cos hi | cos lo | sin hi | sin lo] of eight 16-bit values each, and go straight
// from global memory into LDS.  In 3-D the row operand is the product of the y and z
// factors, tables of FP32 cosines and sines multiplied and split on chip.
//
// A block is eight waves, two per SIMD, with different roles: waves 0-3 only read fragments and
// issue matrix products, waves 4-7 only fill LDS stages of 16 modes, up to three stages ahead
// (four stage buffers, one barrier per stage).  The vector work of the row product (about 90
// instructions per 64 rows and octet) then runs beside the other waves' matrix products instead
// of between them, and the matrix waves, whose next fragments are always ready, read half a
// stage ahead.
//
// What bounds it: 256^3 x 4,096 modes take 0.36-0.44 ms in k_fold, box to box and as the chip warms.  By
// the counters the matrix cores are busy 53% of the cycles, at the 1.86 GHz that the chip holds, and
// a third of that beside vector work, 3.1 instructions for each of their own; no bank conflicts.
// One barrier for all eight waves after loading, splitting and multiplying in turn (no roles) ran at
// 0.60 ms.
// With few modes the stores bound it: four waves write 32,768 cells, and a 64-bit index, bounds and
// three pointer tests per cell took 7 us of every block's time (256 x 256 x 64 modes: 16.4 us, 9.1
// with the addresses and masks below, 6.3 in narrow blocks; 256^3 x 4,096: 422 and 401 in turn on one
// box).
// One call, the separable form with the complex product -> this one: 256^3 0.88 -> 0.42 ms;
// 203 x 171 x 85 x 3,000 modes 0.40 -> 0.087 ms; 128^3 0.17 -> 0.09 ms; 1000 x 500 x 1,024 modes 0.035 ->
// 0.027 ms, x 64 modes 16 us both (the binding's host work); relative error against FP64 2.2e-6 ->
// 7.6e-7 on the ragged grid.  (The hardware cosine in the tables would add 10% to the error.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "grf_internal.h"

namespace grf {

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));

constexpr int kFs = 16;           // modes per stage
constexpr int kTm = 2;            // modes per thread of the table kernel
constexpr int kTabRows = 256 * kTm / 8;  // axis points of a block's pass
constexpr int kRowB = 4 * kFs * 2;  // LDS bytes of one operand row: cos hi, cos lo, sin hi, sin lo

template <bool BF>
__device__ __forceinline__ f32x16 mma(uint4 a, uint4 b, f32x16 c)
{
    if constexpr (BF)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                       0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0,
                                                      0);
}

// Two values as hi words (rounded to nearest) and their remainders.
template <bool BF>
__device__ __forceinline__ uint32_t split_hi(float v0, float v1, f2& r)
{
    const f2 v = {v0, v1};
    if constexpr (BF) {
        const uint32_t hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, b2));
        r = f2{v0 - __builtin_bit_cast(float, hi << 16), v1 - __builtin_bit_cast(float, hi & 0xffff0000u)};
        return hi;
    } else {
        const uint32_t hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, h2));
        // v - hi, the fp16 operand converted by the instruction (one instead of two)
        float r0, r1;
        asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r0) : "v"(hi), "v"(v0));
        asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r1) : "v"(hi), "v"(v1));
        r = f2{r0, r1};
        return hi;
    }
}

template <bool BF>
__device__ __forceinline__ uint32_t round_pair(f2 r)
{
    if constexpr (BF) return __builtin_bit_cast(uint32_t, __builtin_convertvector(r, b2));
    else return __builtin_bit_cast(uint32_t, __builtin_convertvector(r, h2));
}

// As hi words and lo words (the remainders, rounded).
template <bool BF>
__device__ __forceinline__ void split2(float v0, float v1, uint32_t& hi, uint32_t& lo)
{
    f2 r;
    hi = split_hi<BF>(v0, v1, r);
    lo = round_pair<BF>(r);
}

// The same of FP64 values: the remainders hold what FP32 rounds off as well, half a unit of an fp16
// pair's last place (the sums' errors are 1 to 5% lower for it; the tables take up to a tenth
// longer).  A bf16 pair is 2^7 coarser: there FP32 serves.
template <bool BF>
__device__ __forceinline__ void split2(double v0, double v1, uint32_t& hi, uint32_t& lo)
{
    const float f0 = static_cast<float>(v0), f1 = static_cast<float>(v1);
    f2 r;
    hi = split_hi<BF>(f0, f1, r);
    if constexpr (!BF)
        r += f2{static_cast<float>(v0 - static_cast<double>(f0)), static_cast<float>(v1 - static_cast<double>(f1))};
    lo = round_pair<BF>(r);
}

template <bool BF>
__device__ __forceinline__ void split8(const float (&v)[8], uint4& hi, uint4& lo)
{
    split2<BF>(v[0], v[1], hi.x, lo.x);
    split2<BF>(v[2], v[3], hi.y, lo.y);
    split2<BF>(v[4], v[5], hi.z, lo.z);
    split2<BF>(v[6], v[7], hi.w, lo.w);
}

__device__ __forceinline__ int swz(int r) { return (r ^ (r >> 3)) & 7; }

// Exchanges among the four lanes of a quad (q = lane % 4; all four active, every exchange made by all):
// lane q receives word v[q] of lane CTRL % 4, or word a (q < 2) or b of lane (CTRL >> 2 q) % 4.
template <int CTRL>
__device__ __forceinline__ uint32_t quad(uint32_t v)
{
    return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ uint32_t pick4(const uint32_t (&v)[4], int q)
{
    const uint32_t v0 = quad<CTRL>(v[0]), v1 = quad<CTRL>(v[1]), v2 = quad<CTRL>(v[2]), v3 = quad<CTRL>(v[3]);
    return q & 2 ? (q & 1 ? v3 : v2) : (q & 1 ? v1 : v0);
}
template <int CTRL>
__device__ __forceinline__ uint32_t pick2(float a, float b, int q)
{
    const uint32_t u = quad<CTRL>(__builtin_bit_cast(uint32_t, a)), v = quad<CTRL>(__builtin_bit_cast(uint32_t, b));
    return q & 2 ? v : u;
}

// One field's mode table and where its axis tables go.
struct FoldField {
    const double* zx;
    const double* zy;
    const double* zz;
    const double* phi;
    const double* w;
    double fs[3];
    int64_t n;
    uint4* tb;
    uint4* ty;
    uint4* tz;
};

struct FoldTabs {
    FoldField f0, f1;  // f1: the second field of a pair (blockIdx.z = 1)
    double o[3], h[3];
    int64_t ldp, half, ny, nz;  // nz = 0: no z table
    double nx;
    int64_t bb, by, bz;  // thread blocks of the column, y and z tables
};

// One thread: two modes of one octet and one to sixteen points of one axis (an axis' blocks take its
// points in turn); for the octets blockIdx.y, blockIdx.y + gridDim.y .. (more octets than gridDim.y
// can count: tables of 2^19 modes and more).  Bound by the FP64 phases, sines and cosines; with
// eight modes and one point per thread, 30,000 rows x 2,048 modes took 245 us for 148 now,
// 640 axis points x 4,096 modes 20 for 14.5, small tables 5.7 for 3.6.
// Columns, and the rows of a 2-D grid, are stored split; y and z of a 3-D grid as FP32.
template <bool BF>
__global__ __launch_bounds__(256) void k_fold_tables(FoldTabs a)
{
    constexpr double kInvTwoPi = 0.15915494309189533576888376337251;
    const FoldField f = blockIdx.z ? a.f1 : a.f0;
    int64_t b = blockIdx.x;
    const int axis = b < a.bb ? 0 : (b < a.bb + a.by ? 1 : 2);
    b -= axis == 0 ? 0 : (axis == 1 ? a.bb : a.bb + a.by);
    const int64_t rows = axis == 0 ? a.half : (axis == 1 ? a.ny : a.nz);
    const int q = threadIdx.x & 3;  // this thread's pair of modes in the octet, its quarter of the 64 bytes
    const int64_t i0 = b * kTabRows + (threadIdx.x >> 2);  // (all four lanes of a point have the same)
    const int64_t step = kTabRows * (axis == 0 ? a.bb : (axis == 1 ? a.by : a.bz));
    const double* const z = axis == 0 ? f.zx : (axis == 1 ? f.zy : f.zz);
    const double xc = f.fs[0] * (a.o[0] + 0.5 * a.nx * a.h[0]);
    const bool split = axis == 0 || (axis == 1 && a.nz == 0);
    uint4* const base = axis == 0 ? f.tb : (axis == 1 ? f.ty : f.tz);
    for (int64_t oct = blockIdx.y; oct < a.ldp / 8; oct += gridDim.y) {
        double zj[kTm], ps[kTm], w[kTm];
#pragma unroll
        for (int m = 0; m < kTm; ++m) {
            const int64_t j = oct * 8 + kTm * q + m;
            const bool in = j < f.n;  // modes past n add nothing
            zj[m] = in ? z[j] : 0.0;
            ps[m] = in && axis == 1 ? fma(f.zx[j], xc, f.phi[j] * kInvTwoPi) : 0.0;
            w[m] = !in ? 0.0 : (axis == 1 && f.w ? f.w[j] : 1.0);
        }
        for (int64_t i = i0; i < rows; i += step) {
            const double x = axis == 0 ? f.fs[0] * ((static_cast<double>(i) + 0.5 - 0.5 * a.nx) * a.h[0])
                             : axis == 1 ? f.fs[1] * (a.o[1] + (static_cast<double>(i) + 0.5) * a.h[1])
                                         : f.fs[2] * (a.o[2] + (static_cast<double>(i) + 0.5) * a.h[2]);
            double c[kTm], s[kTm];
#pragma unroll
            for (int m = 0; m < kTm; ++m) {
                const double t = zj[m] * x + ps[m];
                sincospi(2.0 * __builtin_amdgcn_fract(t), &s[m], &c[m]);
                c[m] *= w[m];
                s[m] *= w[m];
            }
            // the four lanes of a point exchange words so that each stores 16 contiguous bytes
            uint4 o;
            if (split) {  // [cos hi | cos lo | sin hi | sin lo], eight 16-bit values each
                uint32_t v[4];
                split2<BF>(c[0], c[1], v[0], v[1]);
                split2<BF>(s[0], s[1], v[2], v[3]);
                o = make_uint4(pick4<0x00>(v, q), pick4<0x55>(v, q), pick4<0xaa>(v, q), pick4<0xff>(v, q));
            } else {  // cosines 0-3, 4-7, sines 0-3, 4-7
                const float c0 = static_cast<float>(c[0]), c1 = static_cast<float>(c[1]);
                const float s0 = static_cast<float>(s[0]), s1 = static_cast<float>(s[1]);
                o = make_uint4(pick2<0x88>(c0, s0, q), pick2<0x88>(c1, s1, q), pick2<0xdd>(c0, s0, q),
                               pick2<0xdd>(c1, s1, q));
            }
            // (y of a 3-D grid: each kind in a plane of its own)
            base[oct * rows * 4 + (!split && axis == 1 ? q * rows + i : i * 4 + q)] = o;
        }
    }
}

// One field's axis tables and outputs.
struct FoldSum {
    const uint4* tb;
    const uint4* ty;
    const uint4* tz;
    float amp;
    float* y;
    float* partial;  // raw sums [slice][nq nx] of a launch whose modes are split, or nullptr
};

struct FoldArgs {
    FoldSum f0, f1;  // f1: the second field of a pair (the second half of the items)
    int64_t nx, half, ny, nz, nq;
    int64_t stages, per;  // 16-mode stages in all and per slice, multiples of 4
    int64_t tiles_i, tiles;      // column tiles; tiles of one slice
    int64_t field_items, items;  // tiles of all slices of one field, of all fields
    float* k;
    uint8_t* ind;
};

typedef __attribute__((address_space(3))) void lds_void;
typedef float raw_f4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(4))) raw_f4 scalar_f4;  // constant memory: read by scalar loads

// 16 bytes per lane from a uniform base plus an unsigned 32-bit byte offset below `bytes`, to LDS
// bytes 16 l .. of `s`.  The buffer form: a pending global_load_lds counts as a flat access, and
// the compiler then makes every later wait of the wave a wait for all its loads.
__device__ __forceinline__ void load_to_lds(const char* base, uint32_t bytes, uint32_t off, char* s)
{
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, static_cast<int>(bytes), 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)s, 16, static_cast<int>(off), 0, 0, 0);
}

// Waits until at most VM vector-memory and LG LDS / scalar operations of the wave are under way (15:
// no wait on those).  The builtin, unlike inline assembly, is seen by the compiler's own
// accounting, which then adds no second wait.
template <int VM, int LG>
__device__ __forceinline__ void wait_counts()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt((VM & 15) | (7 << 4) | (LG << 8) | ((VM >> 4) << 14));
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
}

// A barrier that waits for nothing by itself: each role states what it has to wait for.
__device__ __forceinline__ void bare_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
}

// Block: rows q0 .. q0 + BM - 1, columns i0 .. i0 + BN - 1; four matrix waves (2 x 2), each TM x TN
// tiles of 32 x 32 (two accumulators each), and four operand waves.
template <int TM, int TN, bool BF, bool D3>
__global__ __launch_bounds__(512, 2) void k_fold(FoldArgs a, Epi epi)
{
    constexpr int BM = 64 * TM, BN = 64 * TN;
    constexpr int kA = BM * kRowB, kB = BN * kRowB;  // bytes of one stage
    static_assert(BM == 128, "each operand wave makes 32 rows");
    __shared__ __attribute__((aligned(16))) char sa[4 * kA];
    __shared__ __attribute__((aligned(16))) char sb[4 * kB];
    const int l = threadIdx.x & 63, h = l >> 5, lr = l & 31;
    const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    // Consecutive blocks run on different XCDs, each with its own L2: every XCD takes a run of
    // consecutive work items (slice by slice, columns fastest), whose blocks read the same table
    // stages at the same time.  (gridDim.x is a multiple of 8.)
    const int64_t bid = static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x;
    int64_t item = (bid & 7) * (static_cast<int64_t>(gridDim.y) * (gridDim.x >> 3)) + (bid >> 3);
    if (item >= a.items) return;  // the whole block
    const bool second = item >= a.field_items;
    const FoldSum f = second ? a.f1 : a.f0;
    item -= second ? a.field_items : 0;
    const int64_t slice = item / a.tiles, tile = item - slice * a.tiles;
    const int64_t i0 = tile % a.tiles_i * BN, q0 = tile / a.tiles_i * BM;
    const int64_t s0 = slice * a.per, s1 = min(a.stages, s0 + a.per);
    const int ns = static_cast<int>(s1 - s0);  // a multiple of 4, at least 4

    if (w >= 4) {
        // ---- operand waves.  Stage t: columns by direct loads, issued three stages ahead; rows by
        // direct loads too in 2-D, in 3-D from the y and z factors: fetched into registers four
        // stages ahead, multiplied, split and stored two stages ahead.  Past the last stage the
        // last one is loaded again, into buffers that nothing reads any more.
        const int pw = w - 4;
        constexpr int KB = BN / 32, KA = D3 ? 1 : BM / 32;  // direct-load instructions (8 rows each) per wave
        uint32_t offb[KB], offa[KA];
        int ldb[KB], lda[KA];
        auto source = [&](int rb, int64_t first, int64_t rows) {
            const int r = rb * 8 + (l >> 3);
            const int c = (l & 7) ^ swz(r);  // logical chunk: octet, kind (four lanes read 64 bytes)
            const int64_t i = min(first + r, rows - 1);
            return static_cast<uint32_t>(((c >> 2) * rows + i) * 64 + (c & 3) * 16);
        };
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            const int rb = pw * KB + k;
            offb[k] = source(rb, i0, a.half);
            ldb[k] = rb * 8 * kRowB;
        }
        const char* gb = reinterpret_cast<const char*>(f.tb) + 2 * s0 * a.half * 64;
        const char* ga = reinterpret_cast<const char*>(f.ty) + 2 * s0 * a.ny * 64;
        const char* gz = D3 ? reinterpret_cast<const char*>(f.tz) + 2 * s0 * a.nz * 64 : nullptr;
        const int64_t stepb = 128 * a.half, stepa = 128 * a.ny, stepz = 128 * a.nz;
        // 3-D: this wave makes octet pw % 2 of the rows 64 (pw / 2) + l
        const int row = (pw >> 1) * 64 + l, oct = pw & 1;
        uint32_t offy = 0, offz = 0;
        bool onez = false;  // the wave's rows lie in one z-slice: its z factors are uniform
        if constexpr (D3) {
            const int64_t q = min(q0 + row, a.nq - 1);
            offy = static_cast<uint32_t>(oct * a.ny * 64 + q % a.ny * 16);
            offz = static_cast<uint32_t>((oct * a.nz + q / a.ny) * 64);
            const int64_t za = min(q0 + (pw >> 1) * 64, a.nq - 1) / a.ny, zb = min(q0 + (pw >> 1) * 64 + 63, a.nq - 1) / a.ny;
            onez = za == zb;
            gz += (oct * a.nz + za) * 64;  // (per-lane offsets are taken from the first row's)
            offz -= static_cast<uint32_t>((oct * a.nz + za) * 64);
        } else {
#pragma unroll
            for (int k = 0; k < KA; ++k) {
                const int rb = pw * KA + k;
                offa[k] = source(rb, q0, a.ny);
                lda[k] = rb * 8 * kRowB;
            }
        }
        int left_d = ns - 1, left_f = ns - 1, left_z = ns - 1;  // stages the pointers may still advance
        auto direct = [&](int t) {
            char* const bb = sb + (t & 3) * kB;
#pragma unroll
            for (int k = 0; k < KB; ++k) load_to_lds(gb, static_cast<uint32_t>(stepb), offb[k], bb + ldb[k]);
            gb += left_d > 0 ? stepb : 0;
            if constexpr (!D3) {
                char* const ba = sa + (t & 3) * kA;
#pragma unroll
                for (int k = 0; k < KA; ++k) load_to_lds(ga, static_cast<uint32_t>(stepa), offa[k], ba + lda[k]);
                ga += left_d > 0 ? stepa : 0;
            }
            --left_d;
        };
        struct Four {
            float4 v[4];
        };
        // y factors of one stage: four planes of 16 bytes per row (contiguous over the lanes)
        auto fetch_y = [&](Four& r) {
#pragma unroll
            for (int c = 0; c < 4; ++c) r.v[c] = *reinterpret_cast<const float4*>(ga + c * (a.ny * 16) + offy);
            ga += left_f > 0 ? stepa : 0;
            --left_f;
        };
        // z factors; a uniform and constant address is read by scalar loads
        auto fetch_z = [&](Four& r, auto onez_c) {
            if constexpr (decltype(onez_c)::value) {
                const scalar_f4* z = (const scalar_f4*)gz;
#pragma unroll
                for (int c = 0; c < 4; ++c) r.v[c] = __builtin_bit_cast(float4, z[c]);
            } else {
                const float4* z = reinterpret_cast<const float4*>(gz + offz);
#pragma unroll
                for (int c = 0; c < 4; ++c) r.v[c] = z[c];
            }
            gz += left_z > 0 ? stepz : 0;
            --left_z;
        };
        const int x = swz(row);
        char* const wbase = sa + row * kRowB;
        auto put = [&](int t, const Four& y4, const Four& z4) {
            const float* v = reinterpret_cast<const float*>(y4.v);
            const float* z = reinterpret_cast<const float*>(z4.v);
            float c[8], s[8];
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                c[m] = fmaf(v[m], z[m], -(v[8 + m] * z[8 + m]));
                s[m] = fmaf(v[8 + m], z[m], v[m] * z[8 + m]);
            }
            uint4 o[4];
            split8<BF>(c, o[0], o[1]);
            split8<BF>(s, o[2], o[3]);
            char* const base = wbase + (t & 3) * kA;
#pragma unroll
            for (int kind = 0; kind < 4; ++kind) *reinterpret_cast<uint4*>(base + (((4 * oct + kind) ^ x) << 4)) = o[kind];
        };
        direct(0);
        direct(1);
        direct(2);
        auto stages = [&](auto onez_c) {
            constexpr bool kOne = decltype(onez_c)::value;
            Four y0, y1, z0, z1;
            if constexpr (D3) {
                fetch_y(y0);
                fetch_y(y1);
                fetch_z(z0, onez_c);
                fetch_z(z1, onez_c);
                put(0, y0, z0);
                __builtin_amdgcn_sched_barrier(0);
                fetch_z(z0, onez_c);
                __builtin_amdgcn_sched_barrier(0);
                put(1, y1, z1);
            }
            wait_counts<0, 0>();
            if constexpr (D3) {
                fetch_y(y0);
                __builtin_amdgcn_sched_barrier(0);
                fetch_y(y1);
            }
            bare_barrier();
            // y holds stage t + 2's factors and takes stage t + 4's; zc holds stage t + 2's, zn
            // takes stage t + 3's
            auto stage = [&](int t, Four& y, const Four& zc, Four& zn) {
                if constexpr (D3) {
                    fetch_z(zn, onez_c);
                    __builtin_amdgcn_sched_barrier(0);
                    put(t + 2, y, zc);
                    __builtin_amdgcn_sched_barrier(0);
                    direct(t + 3);
                    __builtin_amdgcn_sched_barrier(0);
                    fetch_y(y);
                    // stage t + 2's direct loads have landed: at most the fetches of the
                    // previous iteration and this one's loads are still under way
                    constexpr int kZ = kOne ? 0 : 4;
                    wait_counts<KB + 8 + kZ, 0>();
                } else {
                    direct(t + 3);
                    wait_counts<KB + KA, 15>();
                }
                bare_barrier();
            };
            for (int t = 0; t < ns; t += 2) {
                stage(t, y0, z0, z1);
                stage(t + 1, y1, z1, z0);
            }
        };
        if (D3 && !onez) stages(std::false_type{});
        else stages(std::true_type{});
        wait_counts<0, 15>();  // no load may land in LDS after the block's end
        return;
    }

    // ---- matrix waves
    const int wm = w >> 1, wn = w & 1;
    f32x16 ae[TM][TN], ao[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                ae[i][j][e] = 0.f;
                ao[i][j][e] = 0.f;
            }
    // Fragments of half a stage: the cosines (kinds 0, 1: hi, lo) or the sines (2, 3).
    struct Frag {
        uint4 a[TM][2], b[TN][2];
    };
    int fa[TM][4], fb[TN][4];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int kind = 0; kind < 4; ++kind) {
            const int r = (wm * TM + i) * 32 + lr;
            fa[i][kind] = r * kRowB + (((4 * h + kind) ^ swz(r)) << 4);
        }
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int kind = 0; kind < 4; ++kind) {
            const int r = (wn * TN + j) * 32 + lr;
            fb[j][kind] = r * kRowB + (((4 * h + kind) ^ swz(r)) << 4);
        }
    auto read = [&](int buf, int half, Frag& g) {
#pragma unroll
        for (int x = 0; x < 2; ++x) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
                g.a[i][x] = *reinterpret_cast<const uint4*>(sa + buf * kA + fa[i][2 * half + x]);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                g.b[j][x] = *reinterpret_cast<const uint4*>(sb + buf * kB + fb[j][2 * half + x]);
        }
    };
    auto mac = [&](const Frag& g, f32x16(&acc)[TM][TN]) {
#pragma unroll
        for (int p = 0; p < 3; ++p)  // hi hi, hi lo, lo hi
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = mma<BF>(g.a[i][p == 2], g.b[j][p == 1], acc[i][j]);
    };
    // the reads of the next half ride along the products of this one
    auto interleave = [&]() {
        constexpr int NR = 2 * (TM + TN), NM = 3 * TM * TN;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
        }
        __builtin_amdgcn_sched_group_barrier(0x008, NM - NR > 0 ? NM - NR : 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    // What the stores need, held in registers from here: loads of the arguments after the last stage
    // would each wait for memory.
    const bool raw = f.partial != nullptr;
    float* y = raw ? f.partial + slice * (a.nq * a.nx) : f.y;
    float* kk = raw ? nullptr : a.k;
    uint8_t* ind = raw ? nullptr : a.ind;
    float amp = raw ? 1.f : f.amp;
    int64_t nx = a.nx;
    asm volatile("" : "+s"(y), "+s"(kk), "+s"(ind), "+v"(amp), "+s"(nx));
    Frag f0, f1;
    bare_barrier();
    read(0, 0, f0);
    for (int t = 0; t < ns; t += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            read(u, 1, f1);
            mac(f0, ae);
            interleave();
            // stage t + u + 1 is complete since the last barrier (past the end: unused values)
            read((u + 1) & 3, 0, f0);
            mac(f1, ao);
            interleave();
            bare_barrier();
        }
    }

    // Output addresses: a uniform 64-bit row base and two 32-bit lane offsets per tile (a cell and its
    // mirror, at most 4 rows of 2^24 cells on), rows past the grid masked by one compare.  (The
    // middle cell of an odd row is its own mirror: B = 0 and O = 0 there, the same value twice.)
    auto store = [&](auto put) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int64_t qt = q0 + (wm * TM + i) * 32;
            const int rows = static_cast<int>(min<int64_t>(32, a.nq - qt));
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int64_t col = i0 + (wn * TN + j) * 32 + lr;
                const int lim = col < a.half ? rows - 4 * h : 0;
                const uint32_t c0 = static_cast<uint32_t>(4 * h * nx + col);
                const uint32_t c1 = static_cast<uint32_t>(4 * h * nx + (nx - 1 - col));
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int r = 8 * (e >> 2) + (e & 3);
                    if (r >= lim) continue;
                    const float ev = ae[i][j][e], ov = ao[i][j][e];
                    put((qt + r) * nx, c0, amp * (ev - ov));
                    put((qt + r) * nx, c1, amp * (ev + ov));
                }
            }
        }
    };
    // One pass per output: pointer tests and the facies loop at each cell would cost as much as the stores
    // (192^3 x 200 modes, K alone: 61 us so, 46 now; Y and K 62, 54).
    if (y) store([&](int64_t row, uint32_t c, float v) { global_ptr(y + row)[c] = v; });
    if (kk)
        store([&](int64_t row, uint32_t c, float v) {
#pragma clang fp contract(off)  // Y rounded before mu is added, as in the per-cell path
            global_ptr(kk + row)[c] = expf(epi.mu + v);
        });
    if (ind)
        store([&](int64_t row, uint32_t c, float v) {
            int facies = 0;
            for (int t = 0; t < epi.nthr; ++t) facies += v > epi.thr[t] ? 1 : 0;
            global_ptr(ind + row)[c] = static_cast<uint8_t>(facies);
        });
}

template <int TM, int TN>
hipError_t launch_tile(const FoldArgs& a0, const Epi& epi, bool bf, int slices, int fields, hipStream_t s)
{
    FoldArgs a = a0;
    a.tiles_i = (a.half + 64 * TN - 1) / (64 * TN);
    a.tiles = a.tiles_i * ((a.nq + 64 * TM - 1) / (64 * TM));
    a.field_items = a.tiles * slices;
    a.items = fields * a.field_items;
    const int64_t gy = (a.items + kMaxGridX - 1) / kMaxGridX;
    if (gy > 65535) return hipErrorInvalidValue;
    const dim3 g(static_cast<unsigned>((((a.items + gy - 1) / gy) + 7) / 8 * 8), static_cast<unsigned>(gy)), b(512);
    if (a.f0.tz) {
        if (bf) hipLaunchKernelGGL((k_fold<TM, TN, true, true>), g, b, 0, s, a, epi);
        else hipLaunchKernelGGL((k_fold<TM, TN, false, true>), g, b, 0, s, a, epi);
    } else {
        if (bf) hipLaunchKernelGGL((k_fold<TM, TN, true, false>), g, b, 0, s, a, epi);
        else hipLaunchKernelGGL((k_fold<TM, TN, false, false>), g, b, 0, s, a, epi);
    }
    return hipGetLastError();
}

}  // namespace

bool fold_default(bool bf, int dim, int64_t nx, int64_t ny, int64_t nz, int64_t n)
{
    // On a tall 2-D grid the y table takes most of the time, and halved columns gain little: in bf16,
    // whose separable tables take no software conversion, the complex form is the faster one there
    // up to about 4e6 table entries and 2e8 terms.  One call in us, complex / folded: 16 x 4096 x 512
    // modes 24.6 / 29.0, 40 x 2000 x 512, 1,024, 2,048 20.1 / 21.9, 25.3 / 27.8, 31.7 / 36.1, 100 x 1500 x
    // 1,024 26.2 / 27.6; past the line 40 x 2000 x 4,096 50 / 46, 100 x 1500 x 2,048 39 / 33, 16 x 4096 x
    // 2,048 54 / 46, 200 x 200 x 4,096 26 / 23.  fp16: 16 x 4096 x 512 32 / 29, 40 x 2000 x 2,048 43 / 36.
    return !bf || dim == 3 || 8 * nx > ny || ny * n > (int64_t(1) << 22) ||
           static_cast<double>(nx * ny * nz) * static_cast<double>(n) >= 2e8;
}

FoldWs fold_ws(int64_t nx, int64_t ny, int64_t nz, int64_t ldp, int dim, bool split, int fields)
{
    FoldWs w;
    const int64_t half = (nx + 1) / 2, nq = ny * nz, C = nq * nx;
    w.ty = align256(size_t(half) * ldp * 8);
    w.tz = w.ty + align256(size_t(ny) * ldp * 8);
    w.partial = w.tz + align256(size_t(dim == 3 ? nz : 0) * ldp * 8);
    // One block per CU at a time (LDS), so the blocks run in rounds of 256: 128 rows x 128 columns (2.3 us
    // per four stages, 9.5 us besides, K's exponentials 6 more) or x 64 (1.9, 7, 3).  Launches of at
    // most half the CUs may split the modes into slices of whole groups of four stages (64 modes); the
    // slices' sums take at most 32 MiB, each slice writes and reads 4 bytes per cell at about 4 TB/s,
    // and the second pass costs 3 us besides but hides K's exponentials.  The width and as many slices as
    // make the sum of these smallest, half of K's part counted.  GPU time of a call in us, 128 / 64 columns:
    // 256 x 256 x 64 x 64 modes 17 / 15, x 256 24 / 21, x 2,048 78 (two slices) / 89; 2048 x 2048 x 1,024 56
    // (two slices) / 49; 203 x 171 x 85 x 256 23 / 20, x 3,000 93 (two slices) / 113; 192^3 x 200 40 / 44, x
    // 4,096 348 / 408; 256^3 x 256 47 / 63, x 4,096 435 / 622.  Slices: 256 x 256 x 64 x 256 39 in two, 24
    // in one; 1500 x 1200 x 475 32 in two, 26 in one.
    constexpr int64_t kCUs = 256, kMaxBytes = int64_t(32) << 20;
    const int64_t quads = ldp / (4 * kFs);
    double best = -1.0;
    for (const bool wide : {true, false}) {
        const int64_t cols = wide ? 128 : 64;
        const int64_t blocks = fields * ((half + cols - 1) / cols) * ((nq + 127) / 128);
        const double stage4 = wide ? 2.32 : 1.88, rest = wide ? 9.5 : 7.0, k = wide ? 3.0 : 1.5;
        const double sums = 8.0 * static_cast<double>(fields * C) / 4e6;
        auto take = [&](int64_t per, double cost) {
            if (best >= 0.0 && cost >= best) return;
            best = cost;
            w.wide = wide;
            w.per = 4 * per;
        };
        take(quads, static_cast<double>((blocks + kCUs - 1) / kCUs) * (static_cast<double>(quads) * stage4 + rest + k));
        const int64_t most = split ? std::min<int64_t>(kCUs / blocks, kMaxBytes / (4 * C)) : 1;
        if (most < 2) continue;
        const auto near = static_cast<int64_t>(std::sqrt(static_cast<double>(quads) * sums / stage4));
        for (int64_t per = std::max(near, (quads + most - 1) / most), i = 0; i < 2; ++per, ++i) {
            const int64_t sl = (quads + per - 1) / per;
            if (sl > 1) take(per, static_cast<double>(per) * stage4 + rest + static_cast<double>(sl) * sums + 3.0);
        }
    }
    w.slices = static_cast<int>((4 * quads + w.per - 1) / w.per);
    w.split_bytes = w.slices > 1 ? align256(sizeof(float) * size_t(w.slices) * size_t(C)) : 0;
    return w;
}

static FoldField fold_field(const DirectGrid& d, const FoldWs& w, void* ws)
{
    char* const base = static_cast<char*>(ws);
    return {d.zx, d.zy, d.zz, d.phi, d.w, {d.fs[0], d.fs[1], d.fs[2]}, d.n, reinterpret_cast<uint4*>(base),
            reinterpret_cast<uint4*>(base + w.ty), d.dim == 3 ? reinterpret_cast<uint4*>(base + w.tz) : nullptr};
}

static FoldSum fold_sum(const DirectGrid& d, const FoldWs& w, void* ws)
{
    const FoldField f = fold_field(d, w, ws);
    return {f.tb, f.ty, f.tz, d.amp, d.y,
            w.slices > 1 ? reinterpret_cast<float*>(static_cast<char*>(ws) + w.partial) : nullptr};
}

// The tables of one field, or of two on the same grid (d2 not null) by one launch.
static hipError_t fold_tables(const DirectGrid& d, const DirectGrid* d2, int64_t ldp, bool bf, const FoldWs& w,
                              void* ws, void* ws2, hipStream_t s)
{
    FoldTabs t{};
    t.f0 = fold_field(d, w, ws);
    if (d2) t.f1 = fold_field(*d2, w, ws2);
    for (int a = 0; a < 3; ++a) {
        t.o[a] = d.o[a];
        t.h[a] = d.h[a];
    }
    t.ldp = ldp;
    t.half = (static_cast<int64_t>(d.nx) + 1) / 2;
    t.ny = d.ny;
    t.nz = d.dim == 3 ? d.nq / d.ny : 0;
    t.nx = static_cast<double>(d.nx);
    const int64_t octs = ldp / 8, span = t.half + t.ny + t.nz;
    // about 1,024 blocks where there is that much work: more points per thread share its mode's loads
    const int64_t reps = std::max<int64_t>(1, std::min<int64_t>(16, span * octs / (kTabRows * 1024)));
    const int64_t per = kTabRows * reps;
    t.bb = (t.half + per - 1) / per;
    t.by = (t.ny + per - 1) / per;
    t.bz = (t.nz + per - 1) / per;
    const int64_t tb = t.bb + t.by + t.bz;  // axes are at most 2^24 long
    const dim3 tg(static_cast<unsigned>(tb), static_cast<unsigned>(std::min<int64_t>(octs, 65535)), d2 ? 2 : 1);
    if (bf) hipLaunchKernelGGL(k_fold_tables<true>, tg, dim3(256), 0, s, t);
    else hipLaunchKernelGGL(k_fold_tables<false>, tg, dim3(256), 0, s, t);
    return hipGetLastError();
}

// Their contraction, likewise.
static hipError_t fold_sums(const DirectGrid& d, const DirectGrid* d2, int64_t ldp, bool bf, const Epi& epi,
                            const FoldWs& w, void* ws, void* ws2, hipStream_t s)
{
    FoldArgs a{};
    a.f0 = fold_sum(d, w, ws);
    if (d2) a.f1 = fold_sum(*d2, w, ws2);
    a.nx = d.nx;
    a.half = (static_cast<int64_t>(d.nx) + 1) / 2;
    a.ny = d.ny;
    a.nz = d.dim == 3 ? d.nq / d.ny : 0;
    a.nq = d.nq;
    a.stages = ldp / kFs;
    a.per = w.per;
    a.k = d.k;
    a.ind = d.ind;
    return w.wide ? launch_tile<2, 2>(a, epi, bf, w.slices, d2 ? 2 : 1, s)
                  : launch_tile<2, 1>(a, epi, bf, w.slices, d2 ? 2 : 1, s);
}

hipError_t launch_fold(const DirectGrid& d, int64_t ldp, bool bf, const Epi& epi, void* ws, bool split, hipStream_t s)
{
    const FoldWs w = fold_ws(d.nx, d.ny, d.nq / d.ny, ldp, d.dim, split, 1);
    hipError_t e = fold_tables(d, nullptr, ldp, bf, w, ws, nullptr, s);
    if (e != hipSuccess) return e;
    TimedScope scope(s);  // the contraction and the slice sums
    e = fold_sums(d, nullptr, ldp, bf, epi, w, ws, nullptr, s);
    if (e != hipSuccess || w.slices == 1) return e;
    return launch_points_reduce(reinterpret_cast<float*>(static_cast<char*>(ws) + w.partial), w.slices, d.nq * d.nx,
                                d.amp, epi, d.y, d.k, d.ind, s);
}

hipError_t launch_fold_pair(const DirectGrid& d1, const DirectGrid& d2, int64_t ldp, bool bf, void* ws1, void* ws2,
                            FoldPair* out, std::optional<TimedScope>* timed, hipStream_t s)
{
    const FoldWs w = fold_ws(d1.nx, d1.ny, d1.nq / d1.ny, ldp, d1.dim, true, 2);
    *out = {nullptr, nullptr, w.slices};
    if (w.slices > 1) {
        out->p1 = reinterpret_cast<float*>(static_cast<char*>(ws1) + w.partial);
        out->p2 = reinterpret_cast<float*>(static_cast<char*>(ws2) + w.partial);
    }
    const hipError_t e = fold_tables(d1, &d2, ldp, bf, w, ws1, ws2, s);
    if (e != hipSuccess) return e;
    timed->emplace(s);
    return fold_sums(d1, &d2, ldp, bf, Epi{}, w, ws1, ws2, s);
}

}  // namespace grf
