// Kernels of the learned closure for gfx950: periodic 3x3x3 convolutions on
// BF16 MFMA (v_mfma_f32_16x16x32_bf16, FP32 accumulate) and the small
// elementwise / reduction kernels around them.
//
// Convolution as an implicit GEMM, D[co][cell] = sum_K A[co][K] B[K][cell],
// K = (offset o, input channel ci) flattened as o * CIN + ci, 32 per MFMA.
// MFMA 16x16x32 operand layout (wave64): lane l holds A[l%16][8(l/16)+e],
// B[8(l/16)+e][l%16] (e = 0..7) and D[4(l/16)+e][l%16] (e = 0..3).
//  * A: weights, repacked once per weight update into exactly that layout
//    (one 16-byte load per lane per K step);
//  * B: activations, channel-last x[cell][CIN]: the 8 K values of a lane are
//    8 consecutive channels of one shifted cell (one 16-byte load);
//  * D: 4 consecutive output channels of one cell per lane.
// A workgroup computes tiles of cells x all output channels from an LDS copy
// of the tile's input halo.  dgrad is the same kernel on the gradient with
// the weights flipped (o -> 26 - o) and transposed (ci <-> co), with the ReLU mask of
// the forward activation fused in the epilogue.
//
// wgrad, dW[o][ci][co] = sum_cell x[cell + d(o)][ci] dy[cell][co], has K =
// cells and reads the same channel-last activations through transposing LDS
// reads.  Persistent workgroups write partial sums, which are added in a
// fixed order (deterministic).
//
// Requirements: nx, ny, nz multiples of 32 (the tiles: 16 x 4 x 4 or 8 cells
// for forward / dgrad, 32 x 4 x 2 for wgrad), fewer than 2^31 cells.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <type_traits>

#include "closure_kernels.h"

namespace mhd {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f4;

// bf16 rounding to nearest even (v_cvt_pk_bf16_f32 converts two at a time)
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ uint32_t f2bf2(float lo, float hi)
{
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf2;
    return __builtin_bit_cast(uint32_t, bf2{ (__bf16)lo, (__bf16)hi });
}
__device__ __forceinline__ float bf2f(uint16_t b) { return __builtin_bit_cast(float, (uint32_t)b << 16); }

__device__ __forceinline__ bf16x8 as_bf8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }
__device__ __forceinline__ uint4 ld16(const uint16_t* p) { return *reinterpret_cast<const uint4*>(p); }

__device__ __forceinline__ int wrap1(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// (i, j, k) of cell c = i + nx (j + ny k), 32-bit arithmetic (fewer than 2^31 cells)
__device__ __forceinline__ void cell_ijk(unsigned c, int nx, int ny, int& i, int& j, int& k)
{
    const unsigned q = c / (unsigned)nx;
    i = (int)(c - q * (unsigned)nx);
    const unsigned k_ = q / (unsigned)ny;
    j = (int)(q - k_ * (unsigned)ny);
    k = (int)k_;
}

// ---------------------------------------------------------------------------
// weight packing
// ---------------------------------------------------------------------------
// Wp[s][m][lane][e] = W'[o][ci][co] with K = 32 s + 8 (lane/16) + e,
// o = K / cin, ci = K % cin, co = 16 m + lane % 16; zero outside.  flip:
// W'[o][ci][co] = W[26 - o][co][ci] (dgrad of a layer with weights W[27][co][ci]).
__global__ void pack_weights_kernel(const float* __restrict__ w, int cin, int cout, int flip,
                                    uint16_t* __restrict__ wp)
{
    const int ks = (27 * cin + 31) / 32, mb = (cout + 15) / 16;
    const int total = ks * mb * 64 * 8;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < total; t += gridDim.x * blockDim.x) {
        const int e = t & 7, lane = (t >> 3) & 63, m = (t >> 9) % mb, s = (t >> 9) / mb;
        const int K = 32 * s + 8 * (lane >> 4) + e;
        const int o = K / cin, ci = K % cin, co = 16 * m + (lane & 15);
        float v = 0.0f;
        if (o < 27 && co < cout)
            v = flip ? w[((size_t)(26 - o) * cout + co) * cin + ci] : w[((size_t)o * cin + ci) * cout + co];
        wp[t] = f2bf(v);
    }
}

hipError_t launch_pack_weights(const float* w, int cin, int cout, int flip, uint16_t* wp, hipStream_t s)
{
    hipLaunchKernelGGL(pack_weights_kernel, dim3(64), dim3(256), 0, s, w, cin, cout, flip, wp);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// forward / dgrad convolution
// ---------------------------------------------------------------------------

// Persistent workgroups, one per CU.  A wave keeps its weights in registers
// for the whole launch (a workgroup per tile read 55 KiB of them per wave and
// tile, as many L1 cycles as MFMA cycles), and the next tile's halo is on its
// way through registers to the second of two LDS buffers while a tile is
// multiplied (one barrier per tile).  With 32 input channels a workgroup is 4
// waves, one per SIMD with all its registers: a halo row read from LDS feeds
// all 32 output channels of a z plane (54 weight fragments, 216 registers;
// tile 16 x 4 x 4 cells), or the 8 of two planes (16 x 4 x 8), whose 16 MFMA
// rows are those of two neighbouring rows y (a pair of output rows has 4 input
// rows, so 36 products where one row per accumulator takes 54; 36 fragments
// with the absent offsets zero).  With 8 input channels (7 fragments of four
// offsets each) it is 8 waves: bound by memory, not by products.
// 128^3 in us (workgroup per tile -> persistent, 8 waves, loads and epilogue
// before and after the products -> now): 32 -> 32 channels 151 -> 135 -> 114,
// 32 -> 8 99 -> 83 -> 62, 8 -> 32 64 -> 58 -> 49.  Gated forward with all
// passes, of the last two forms: 96 x 64 x 64 83.5 -> 81.5, 64^3 65.5 -> 66.2,
// 32^3 36.3 -> 38.6 (a tile or less per workgroup: the longer start is not
// paid back).  The products alone with their LDS reads take 75, 36 and
// 31 (all 116 GFLOP of the first at 1.5 PFLOP/s); the halo's way through
// registers costs 25, the epilogue 10, stores in flight 10.
// A wave's MFMA columns are the 16 cells of a row, lane r the cell x.  The
// input halo is staged in LDS once per tile, rows of 20 cells.
// A B read has 16 lanes on 16 consecutive cells reading the same 16-byte
// chunk; with 64-byte cells (CIN = 32) the chunks of cells h and h + 4 would
// share banks, so chunk q of cell h is stored at position q ^ 2 ((h >> 2) &
// 1): any 8 consecutive cells then fall on distinct bank groups (measured on
// gfx950: a lane stride that is an odd multiple of 32 bytes modulo 256, or
// this swizzle, is conflict-free; 64 or 80 bytes costs two passes).  With
// rows of 20 cells the swizzle only flips from row to row, so a lane needs
// two base addresses and every row is an immediate offset.
constexpr int CT_X = 16, CT_Y = 4;
constexpr int CH_X = CT_X + 2, CH_Y = CT_Y + 2;
constexpr int CL_X = 20;         // LDS cells per halo row (18 used)
constexpr int CONV_WGS = 256;

template <int CIN, int COUT>
struct ConvShape {
    static constexpr int WAVES = CIN == 32 ? 4 : 8, THREADS = 64 * WAVES;
    static constexpr bool FOLD = CIN == 32 && COUT == 8;   // MFMA rows hold 8 channels of two rows y
    static constexpr int MB = (COUT + 15) / 16;            // 16-row blocks of output channels
    static constexpr int MBW = CIN == 32 ? MB : 1;         // of them in a wave
    static constexpr int ZW = FOLD ? 2 : 1;                // z planes of a wave
    static constexpr int TZ = WAVES * MBW / MB * ZW;       // of a tile
    static constexpr int CELLS = CH_X * CH_Y * (TZ + 2);   // halo cells
    static constexpr int LDS = CL_X * CH_Y * (TZ + 2) * CIN;   // bf16 values of a buffer
    static constexpr int PARTS = CIN / 8;                  // 16-byte pieces per cell
    static constexpr int KS = FOLD ? 36 : (27 * CIN + 31) / 32;    // weight fragments per 16 rows
    static constexpr int NB = FOLD ? CT_Y / 2 : CT_Y;      // accumulators per plane and 16 rows
    static constexpr int NA = ZW * MBW * NB;
    static constexpr int FILL = (CELLS * PARTS + THREADS - 1) / THREADS;
    // tiles the loads run ahead: to be filled at the end of this one, or of
    // the next, each piece loaded when the one before has left its registers
    // (128^3, 32 -> 8 channels 69 -> 63 us; 32 -> 32 has no registers for it)
    static constexpr int AHEAD = FOLD ? 2 : 1;
    static constexpr int PHASES = CIN == 32 ? (ZW + 2) * CH_Y : KS;    // parts a tile's products are taken in
};
// position (in 8-bf16 chunks) of chunk q of halo cell h
template <int CIN>
__device__ __forceinline__ int conv_chunk(int h, int q) { return CIN == 32 ? (q ^ (((h >> 2) & 1) << 1)) : q; }

// Visit order of the tiles.  A tile's halo is 2.1 to 2.5 times its cells, so
// what neighbouring tiles read in common has to come from L2, and each XCD has
// its own (the hardware deals workgroups round-robin over the 8): XCD k takes
// the k-th eighth of the visits, which go in columns of CONV_YG tiles along y
// through z with all x tiles of a z in turn, so that the planes shared with
// the next z are read again a few dozen visits later.  (Grids are multiples of
// 32: the number of tiles is a multiple of 16 and ty of 8.)
constexpr int CONV_YG = 4;
// A visit o is x + tx (y % YG + YG (z + tz (y / YG))), tile coordinates
// stepped by a fixed number of visits with carries (a division by tx or tz is
// a chain of a dozen scalar instructions).
struct ConvVisit {
    int x, yl, z, yh;
};
__device__ __forceinline__ ConvVisit conv_visit(int o, int tx, int tz)
{
    const int q = o / tx, w = q / CONV_YG;
    return ConvVisit{ o % tx, q % CONV_YG, w % tz, w / tz };
}
__device__ __forceinline__ ConvVisit conv_next(ConvVisit v, ConvVisit d, int tx, int tz)
{
    v.x += d.x;
    int c = v.x >= tx;
    v.x -= c ? tx : 0;
    v.yl += d.yl + c;
    c = v.yl >= CONV_YG;
    v.yl -= c ? CONV_YG : 0;
    v.z += d.z + c;
    c = v.z >= tz;
    v.z -= c ? tz : 0;
    v.yh += d.yh + c;
    return v;
}

// the fragment of cells x from those of x - 1 and x + 1 (16 lanes of a K
// chunk): lanes 0 - 11 take the next lane's x - 1, lanes 12 - 15 the previous
// lane's x + 1
__device__ __forceinline__ bf16x8 between(bf16x8 left, bf16x8 right)
{
    typedef __attribute__((__vector_size__(4 * sizeof(int)))) int i4;
    const i4 l = __builtin_bit_cast(i4, left), r = __builtin_bit_cast(i4, right);
    i4 o;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int a = __builtin_amdgcn_mov_dpp(l[q], 0x101, 0xf, 0x7, false);              // row_shl:1, the others follow
        o[q] = __builtin_amdgcn_update_dpp(a, r[q], 0x111, 0xf, 0x8, false);               // row_shr:1
    }
    return __builtin_bit_cast(bf16x8, o);
}

// two bf16 values, each kept where the mask's value is positive
__device__ __forceinline__ uint32_t masked2(uint32_t v, uint32_t mk)
{
    const uint32_t lo = bf2f((uint16_t)(mk & 0xffff)) > 0.0f ? v & 0xffffu : 0u;
    const uint32_t hi = bf2f((uint16_t)(mk >> 16)) > 0.0f ? v & 0xffff0000u : 0u;
    return lo | hi;
}

#define INLINE __attribute__((always_inline))   // (a lambda called outright keeps what it captures in memory)
// Offset: an unsigned type that counts the 16-byte pieces of the input
template <int CIN, int COUT, int EPI, typename Offset>
__global__ void __launch_bounds__((ConvShape<CIN, COUT>::THREADS), (ConvShape<CIN, COUT>::WAVES / 4)) conv3d_kernel(ConvArgs A)
{
    using S = ConvShape<CIN, COUT>;
    constexpr int THREADS = S::THREADS, MBW = S::MBW, ZW = S::ZW, NB = S::NB, NA = S::NA, KS = S::KS, FILL = S::FILL, AHEAD = S::AHEAD;
    constexpr int PIECES = S::CELLS * S::PARTS;
    constexpr bool FOLD = S::FOLD, BIAS = EPI == EPI_BIAS_RELU || EPI == EPI_BIAS_F32 || EPI == EPI_CLOSURE;
    // 32 output channels in bf16 leave through LDS (two buffers, so that the
    // barrier of a tile is enough): 4 chunks of 16 bytes per cell, chunk q of
    // cell c at q ^ ((c >> 2) & 3), which spreads 16 cells over the banks
    constexpr bool STAGED = EPI == EPI_BIAS_RELU || EPI == EPI_MASK;
    static_assert(!STAGED || COUT == 32, "the layers with 8 output channels leave in FP32");
    constexpr int OUT = STAGED ? CT_X * CT_Y * S::TZ * COUT : 8;
    constexpr int CHUNKS = STAGED ? OUT / 8 / THREADS : 1;
    __shared__ __align__(16) uint16_t tiles[2 * S::LDS];
    __shared__ __align__(16) uint16_t stage[2 * OUT];
    __shared__ double wave_sum[EPI == EPI_CLOSURE ? S::WAVES : 1][8];

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane >> 4, r = lane & 15;
    const int m0 = (wave * MBW) % S::MB, wz = wave * MBW / S::MB * ZW;     // first block and plane of the wave
    const int nx = A.n[0], ny = A.n[1], nz = A.n[2];
    const uint16_t* __restrict__ x = A.x;
    const uint4* __restrict__ wp = reinterpret_cast<const uint4*>(A.wp);

    bf16x8 a[KS][MBW];
    int rows[2] = { r < 8 ? -1 : 0, r < 8 ? 0 : -1 };       // (opaque: no branch around the loads)
    asm volatile("" : "+v"(rows[0]), "+v"(rows[1]));
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int m = 0; m < MBW; ++m) {
            if constexpr (FOLD) {
                // fragment (dz, j, dx): rows 0 - 7 the weights of dy = j, rows
                // 8 - 15 those of dy = j - 1 (input row 2 P + j to output rows
                // 2 P and 2 P + 1)
                const int dz = s / 12, j = s / 3 % 4, dx = s % 3, dy = j - (r >> 3);
                uint4 v = wp[(dz * 9 + (dy < 0 ? 0 : dy > 2 ? 2 : dy) * 3 + dx) * 64 + (lane & ~8)];
                if (j == 0 || j == 3) {
                    const int keep = rows[j / 3];
                    v = make_uint4(v.x & keep, v.y & keep, v.z & keep, v.w & keep);
                }
                a[s][m] = as_bf8(v);
            } else {
                a[s][m] = as_bf8(wp[((size_t)s * S::MB + m0 + m) * 64 + lane]);
            }
        }
    // the lane's 4 output channels of block m; where it holds none of COUT = 8
    // (rows 8 - 15 without FOLD) it stores nothing
    auto channel = [&](int m) INLINE { return FOLD ? 4 * (g & 1) : 16 * (m0 + m) + 4 * g; };
    float bias[MBW][4];
#pragma unroll
    for (int m = 0; m < MBW; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e) bias[m][e] = BIAS && channel(m) + e < COUT ? A.bias[channel(m) + e] : 0.0f;
    // visits o, o + stride, ... below end of this workgroup's XCD
    const int tx = nx / CT_X, ty = ny / CT_Y, tz = nz / S::TZ, per = (tx * ty * tz) >> 3;
    const int stride = gridDim.x >> 3, end = ((blockIdx.x & 7) + 1) * per;
    int o = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (o >= end) return;
    ConvVisit at = conv_visit(o, tx, tz);
    const ConvVisit hop = conv_visit(stride, tx, tz);

    // piece q of halo cell h per thread and round, consecutive threads on
    // consecutive pieces (contiguous along x in global memory): its LDS place
    // (in pieces) with the faces of the halo it lies on (bits 14 + 2 axis lower, 15 + 2
    // axis upper; one register per round, opaque below, or the compiler keeps
    // every derived value across the loop and spills), and its offset from
    // the halo's first cell, unwrapped
    int place[FILL];
    Offset delta[FILL], src[FILL];                          // in pieces, modulo the type's range
    typedef __attribute__((__vector_size__(4 * sizeof(int)))) int i4;
    i4 fv[FILL];
    const Offset wx = (Offset)S::PARTS * nx, wy = wx * ny, wz_ = wy * nz;      // periods
    constexpr int HOP = THREADS / S::PARTS;                 // cells from round to round
    const int h0 = threadIdx.x / S::PARTS, q = threadIdx.x % S::PARTS;
    int hx = h0 % CH_X, hy = h0 / CH_X % CH_Y, hz = h0 / (CH_X * CH_Y);
    Offset off = (Offset)(S::PARTS * hx + q) + wx * hy + wy * hz;
#pragma unroll
    for (int f = 0; f < FILL; ++f) {
        if (f + 1 == FILL && THREADS * FILL > PIECES && (int)threadIdx.x + THREADS * f >= PIECES) {
            // threads past the last piece repeat the first ones (the same
            // values to the same place), so that no load sits in a branch
            const int h = (threadIdx.x + THREADS * f - PIECES) / S::PARTS;
            hx = h % CH_X; hy = h / CH_X % CH_Y; hz = h / (CH_X * CH_Y);
            off = (Offset)(S::PARTS * hx + q) + wx * hy + wy * hz;
        }
        const int hl = (hz * CH_Y + hy) * CL_X + hx;
        place[f] = (hl * S::PARTS + conv_chunk<CIN>(hl, q)) | (hx == 0) << 14 | (hx == CH_X - 1) << 15 | (hy == 0) << 16 |
                   (hy == CH_Y - 1) << 17 | (hz == 0) << 18 | (hz == S::TZ + 1) << 19;
        delta[f] = off;
        // the next round's cell, without divisions
        off += (Offset)(S::PARTS * (HOP % CH_X)) + wx * (HOP / CH_X % CH_Y) + wy * (HOP / (CH_X * CH_Y));
        hx += HOP % CH_X;
        hy += HOP / CH_X % CH_Y;
        hz += HOP / (CH_X * CH_Y);
        if (hx >= CH_X) { hx -= CH_X; ++hy; off += wx - S::PARTS * CH_X; }
        if (hy >= CH_Y) { hy -= CH_Y; ++hz; off += wy - wx * CH_Y; }
    }
    // where the pieces of a tile's halo are; its first cell
    auto aim = [&](const ConvVisit& v) INLINE {
        const int by = v.yh * CONV_YG + v.yl;
        const long c0 = (long)(v.x * CT_X) + (long)nx * ((long)(by * CT_Y) + (long)ny * (v.z * S::TZ));
        const Offset first = (Offset)(c0 * S::PARTS) - (S::PARTS + wx + wy);
#pragma unroll
        for (int f = 0; f < FILL; ++f) src[f] = first + delta[f];
        // a tile at a face of the grid: the pieces beyond it, one period back
        auto wrap = [&](int bit, Offset period) INLINE {
#pragma unroll
            for (int f = 0; f < FILL; ++f) {
                int p = place[f];
                asm volatile("" : "+v"(p));
                src[f] += (Offset)0 - (Offset)(p >> bit & 1) & period;
            }
        };
        if (v.x == 0) wrap(14, wx);
        if (v.x + 1 == tx) wrap(15, 0 - wx);
        if (by == 0) wrap(16, wy);
        if (by + 1 == ty) wrap(17, 0 - wy);
        if (v.z == 0) wrap(18, wz_);
        if (v.z + 1 == tz) wrap(19, 0 - wz_);
        return c0;
    };
    auto load = [&](int f) INLINE { fv[f] = reinterpret_cast<const i4*>(x)[src[f]]; };
    auto fill = [&](uint16_t* tile, int f) INLINE {
        int p = place[f];
        asm volatile("" : "+v"(p));
        *reinterpret_cast<i4*>(tile + 8 * (p & 0x3fff)) = fv[f];
    };

    // All waves of the CU are in the same phase between two barriers, so what
    // a wave does outside its products is time without products.  Each tile's
    // products are therefore taken in PHASES parts, and between them go: the
    // loads of the next halo (first), the epilogue of the tile before (acc_old,
    // an accumulator per phase: to LDS where STAGED, else to memory), the
    // stores of the tile before that one (STAGED), and the next halo's way to
    // LDS (last).
    f4 acc[NA], acc_old[NA];                                // [plane][block][row or pair of rows]
    float gate[NA];                                         // EPI_CLOSURE, of acc_old's cells
    double sum[4] = { 0, 0, 0, 0 };                         // EPI_CLOSURE: of the lane's 4 channels
    bool nan = false;                                       // FOLD: a NaN among the accumulators so far
    uint4 mask[CHUNKS], chunk[CHUNKS];
    long c_fetched = 0, c_now, c_old = 0, c_out = 0;        // first cells: of fv, of acc, of acc_old, staged

    // the cell of the tile that the lane holds of accumulator u
    auto row = [&](int u) INLINE { return FOLD ? 2 * (u % NB) + (g >> 1) : u % NB; };
    auto plane_of = [&](int u) INLINE { return wz + u / (NB * MBW); };
    auto cell = [&](long c0, int u) INLINE { return c0 + r + (long)nx * (row(u) + (long)ny * plane_of(u)); };
    auto epilogue = [&](int u, uint16_t* st) INLINE {
        const int m = u / NB % MBW, co0 = channel(m);
        if (co0 >= COUT) return;
        const long c = cell(c_old, u);
        if (FOLD && EPI != EPI_CLOSURE)
            nan = nan || __builtin_isunordered(acc_old[u][0], acc_old[u][1]) || __builtin_isunordered(acc_old[u][2], acc_old[u][3]);
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = acc_old[u][e];
            if (BIAS) v[e] += bias[m][e];
            if (EPI == EPI_CLOSURE) {
                if (A.gate) v[e] *= gate[u];
                sum[e] += (double)v[e];
            }
            if (EPI == EPI_BIAS_RELU) v[e] = fmaxf(v[e], 0.0f);
        }
        if constexpr (STAGED) {
            const int cl = (plane_of(u) * CT_Y + row(u)) * CT_X + r, q = co0 >> 3;
            *reinterpret_cast<uint2*>(st + cl * COUT + 8 * (q ^ ((cl >> 2) & 3)) + (co0 & 4)) =
                make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
        } else {
            *reinterpret_cast<float4*>(A.yf + (size_t)c * COUT + co0) = make_float4(v[0], v[1], v[2], v[3]);
        }
    };
    auto load_gate = [&]() INLINE {
        if constexpr (EPI == EPI_CLOSURE)
#pragma unroll
            for (int u = 0; u < NA; ++u) gate[u] = A.gate ? A.gate[cell(c_old, u)] : 1.0f;
    };
    // STAGED: consecutive threads store consecutive chunks, 1 KiB per wave and row
    auto staged_cell = [&](int i, int& cl, int& q) INLINE {
        const int p = threadIdx.x + THREADS * i;
        cl = p >> 2;
        q = p & 3;
        return c_out + cl % CT_X + (long)nx * ((cl / CT_X) % CT_Y + (long)ny * (cl / (CT_X * CT_Y)));
    };
    auto load_mask = [&]() INLINE {
        if constexpr (STAGED && EPI == EPI_MASK)
#pragma unroll
            for (int i = 0; i < CHUNKS; ++i) {
                int cl, q;
                const long c = staged_cell(i, cl, q);
                mask[i] = ld16(A.mask + (size_t)c * COUT + 8 * q);
            }
    };
    auto load_staged = [&](const uint16_t* st, int i) INLINE {
        int cl, q;
        staged_cell(i, cl, q);
        return *reinterpret_cast<const uint4*>(st + cl * COUT + 8 * (q ^ ((cl >> 2) & 3)));
    };
    auto store_staged = [&](uint4 v, int i) INLINE {
        int cl, q;
        const long c = staged_cell(i, cl, q);
        if constexpr (EPI == EPI_MASK) {
            v.x = masked2(v.x, mask[i].x); v.y = masked2(v.y, mask[i].y);
            v.z = masked2(v.z, mask[i].z); v.w = masked2(v.w, mask[i].w);
        }
        *reinterpret_cast<uint4*>(A.yb + (size_t)c * COUT + 8 * q) = v;
    };

    // products of the tile in buffer buf, and what goes between them; old,
    // out, fetch: there is a tile before, one before that, one to load
    auto work = [&](int buf, auto old, auto out, auto fetch) INLINE {
        constexpr bool FETCH = decltype(fetch)::value;
        const uint16_t* const tile = tiles + buf * S::LDS;
        long c_next = 0;
        auto between_products = [&](int k) INLINE {
            constexpr int ROW0 = EPI == EPI_CLOSURE ? 5 : 1;        // later where the gate is loaded first
            constexpr int STORE = CIN == 32 ? 2 : 1, FILLS = AHEAD == 2 ? 1 : CIN == 32 ? 2 : FILL;
            if (k == 0) {
                if (STAGED && out) load_mask();
                if (old) load_gate();
                if constexpr (FETCH) c_next = aim(at);
            }
            if constexpr (FETCH && AHEAD == 1)
#pragma unroll
                for (int f = 0; f < FILL; ++f)
                    if (k == f / FILLS) load(f);
            if (k >= ROW0 && k < ROW0 + NA)
                if (old) epilogue(k - ROW0, stage + (buf ^ 1) * OUT);
            if (STAGED && out)
#pragma unroll
                for (int i = 0; i < CHUNKS; ++i) {
                    if (k == STORE + 2 * i) chunk[i] = load_staged(stage + buf * OUT, i);
                    if (k == STORE + 2 * i + 1) store_staged(chunk[i], i);
                }
            if constexpr (FETCH)
#pragma unroll
                for (int f = 0; f < FILL; ++f)
                    if (k == S::PHASES - (FILL + FILLS - 1) / FILLS + f / FILLS) {
                        fill(tiles + (buf ^ 1) * S::LDS, f);
                        if constexpr (AHEAD == 2) load(f);
                    }
        };
#pragma unroll
        for (int u = 0; u < NA; ++u) acc[u] = f4{ 0.f, 0.f, 0.f, 0.f };
        if constexpr (CIN == 32) {
            // one offset per K step.  Read offset by offset, every row of the
            // halo would be read from LDS nine times (3 dy, 3 dx), twice the
            // LDS cycles of the MFMA cycles it feeds; here a row is read twice
            // (dx = -1, +1; dx = 0 by lane shifts of the two) and feeds the
            // output rows row - dy of all three dy.  Each accumulator adds its offsets in the order
            // dz, dy, dx.
            const uint16_t* const plane = tile + wz * (CH_Y * CL_X * CIN);
            const uint16_t *leftp[2], *rightp[2];           // lane bases of even and odd rows
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                leftp[p] = plane + r * CIN + 8 * conv_chunk<CIN>(4 * p + r, g);
                rightp[p] = plane + (r + 2) * CIN + 8 * conv_chunk<CIN>(4 * p + r + 2, g);
            }
            auto ld_row = [&](const uint16_t* const (&base)[2], int k) INLINE {    // row k of the wave's three planes
                return as_bf8(*reinterpret_cast<const uint4*>(base[k & 1] + k * (CL_X * CIN)));
            };
            bf16x8 left = ld_row(leftp, 0), right = ld_row(rightp, 0);
#pragma unroll
            for (int k = 0; k < S::PHASES; ++k) {
                const int p = k / CH_Y, in = k % CH_Y;
                bf16x8 left1 = left, right1 = right;
                if (k + 1 < S::PHASES) {                    // the next row, ahead of this one's products
                    left1 = ld_row(leftp, k + 1);
                    right1 = ld_row(rightp, k + 1);
                    __builtin_amdgcn_sched_barrier(0);      // (the scheduler would move them behind)
                }
                const bf16x8 b[3] = { left, between(left, right), right };
                // dx outside: consecutive products go to different accumulators
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                    for (int u = 0; u < NA; ++u) {
                        const int dz = p - u / (NB * MBW), m = u / NB % MBW;
                        const int j = in - (FOLD ? 2 : 1) * (u % NB);       // dy, or the pair's input row
                        if (dz < 0 || dz > 2 || j < 0 || j > (FOLD ? 3 : 2)) continue;
                        acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[(dz * (FOLD ? 4 : 3) + j) * 3 + dx][m], b[dx], acc[u], 0, 0, 0);
                    }
                between_products(k);
                left = left1;
                right = right1;
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            // 4 offsets per K step, one per K chunk g (offset 27 is padding)
            const int hbase = (wz + 1) * (CL_X * CH_Y) + CL_X + (r + 1);
            auto load_b = [&](int s, bf16x8* bv) INLINE {
                const int of = 4 * s + g;
                const int dx = of % 3 - 1, dy = (of / 3) % 3 - 1, dz = of / 9 - 1;
                const int h0 = hbase + dz * (CL_X * CH_Y) + dy * CL_X + dx;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    uint4 v = make_uint4(0, 0, 0, 0);
                    if (of < 27) v = *reinterpret_cast<const uint4*>(tile + (h0 + nb * CL_X) * CIN);
                    bv[nb] = as_bf8(v);
                }
            };
            bf16x8 b_cur[NB];
            load_b(0, b_cur);
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                bf16x8 b_nxt[NB];
                if (s + 1 < KS) load_b(s + 1, b_nxt);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s][0], b_cur[nb], acc[nb], 0, 0, 0);
                between_products(s);
                if (s + 1 < KS)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) b_cur[nb] = b_nxt[nb];
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NA; ++u) acc_old[u] = acc[u];
        c_out = c_old;
        c_old = c_now;
        c_now = AHEAD == 2 ? c_fetched : c_next;
        c_fetched = c_next;
    };
    // the visit loaded next, AHEAD of o: the last one again at the end (unused)
    auto advance = [&](int ahead) INLINE {
        if (o + ahead * stride < end) at = conv_next(at, hop, tx, tz);
    };
    c_now = aim(at);
#pragma unroll
    for (int u = 0; u < NA; ++u) acc_old[u] = f4{ 0.f, 0.f, 0.f, 0.f };
#pragma unroll
    for (int f = 0; f < FILL; ++f) load(f);
    // waited for here: in the loop the wait would take in the halo loads that
    // are to stay in flight over the products
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int m = 0; m < MBW; ++m) asm volatile("" : "+v"(a[s][m]));
#pragma unroll
    for (int m = 0; m < MBW; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e) asm volatile("" : "+v"(bias[m][e]));
    if constexpr (AHEAD == 2) {
        advance(1);
        c_fetched = aim(at);
    }
#pragma unroll
    for (int f = 0; f < FILL; ++f) {
        fill(tiles, f);
        if constexpr (AHEAD == 2) load(f);
    }
    __syncthreads();
    advance(AHEAD);
    // the first tiles have none before them to store (the epilogue of a STAGED
    // one that is not there goes to LDS, where nobody reads it), the last one
    // none after it to load
    constexpr int FIRST = STAGED ? 2 : 1;
    int buf = 0, done = 0;
    auto next = [&]() INLINE {
        ++done;
        buf ^= 1;
        o += stride;
        advance(AHEAD);
    };
#pragma unroll 1
    while (done < FIRST && o + stride < end) {
        work(buf, std::bool_constant<STAGED>(), std::false_type(), std::true_type());
        next();
    }
#pragma unroll 1
    while (o + stride < end) {
        work(buf, std::true_type(), std::true_type(), std::true_type());
        next();
    }
    work(buf, done > 0, done > 1, std::false_type());
    ++done;
    if constexpr (STAGED)
        if (done > 1) {                                     // the last tile but one
            load_mask();
#pragma unroll
            for (int i = 0; i < CHUNKS; ++i) store_staged(load_staged(stage + (buf ^ 1) * OUT, i), i);
        }
    load_gate();
#pragma unroll
    for (int u = 0; u < NA; ++u) epilogue(u, stage + buf * OUT);
    if constexpr (STAGED) {
        __syncthreads();
        c_out = c_old;
        load_mask();
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i) store_staged(load_staged(stage + buf * OUT, i), i);
    }
    // In the folded form a row that only one of the two output rows may see
    // meets zero weights in the other's MFMA rows, and zero times an infinity
    // or a NaN is a NaN, outside its stencil.  So where a workgroup finds a NaN
    // (EPI_CLOSURE: in its sums) it takes all its tiles again, the two output
    // rows one after the other, each with its own input rows and its weights in
    // all 16 MFMA rows.  (Tested for and mended tile by tile, between the
    // products and the barrier, this cost 2.5 us of the 62 at 128^3; by a
    // reduction of its own at the end, 2 us of 70 at 96 x 64 x 64.)
    auto apart = [&]() INLINE {
        o = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
        at = conv_visit(o, tx, tz);
#pragma unroll 1
        for (; o < end; o += stride, at = conv_next(at, hop, tx, tz)) {
            c_old = aim(at);
#pragma unroll
            for (int f = 0; f < FILL; ++f) load(f);
#pragma unroll
            for (int f = 0; f < FILL; ++f) fill(tiles, f);
            __syncthreads();
            const uint16_t* const base = tiles + wz * (CH_Y * CL_X * CIN);
#pragma unroll 1
            for (int half = 0; half < 2; ++half) {
                f4 one[NA];
#pragma unroll
                for (int u = 0; u < NA; ++u) one[u] = f4{ 0.f, 0.f, 0.f, 0.f };
#pragma unroll 1
                for (int k = 0; k < S::PHASES; ++k) {
                    const int p = k / CH_Y, in = k % CH_Y;
                    const bf16x8 left = as_bf8(*reinterpret_cast<const uint4*>(base + (k * CL_X + r) * CIN + 8 * conv_chunk<CIN>(k * CL_X + r, g)));
                    const bf16x8 right = as_bf8(*reinterpret_cast<const uint4*>(base + (k * CL_X + r + 2) * CIN + 8 * conv_chunk<CIN>(k * CL_X + r + 2, g)));
                    const bf16x8 b[3] = { left, between(left, right), right };
#pragma unroll
                    for (int u = 0; u < NA; ++u) {
                        const int dz = p - u / NB, dy = in - 2 * (u % NB) - half;
                        if (dz < 0 || dz > 2 || dy < 0 || dy > 2) continue;
#pragma unroll
                        for (int dx = 0; dx < 3; ++dx)
                            one[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                as_bf8(wp[(dz * 9 + dy * 3 + dx) * 64 + (lane & ~8)]), b[dx], one[u], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int u = 0; u < NA; ++u)
                    if (half == g >> 1) acc_old[u] = one[u];
            }
            load_gate();
#pragma unroll
            for (int u = 0; u < NA; ++u) epilogue(u, nullptr);
            __syncthreads();                            // the tile's buffer is free again
        }
    };
    if constexpr (EPI == EPI_CLOSURE) {
        // the workgroup's channel sums: 16 lanes of a channel, then the waves
        // (every thread has the total of channel threadIdx.x % 8)
        auto totals = [&]() INLINE {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int st = FOLD ? 32 : 8; st > 0; st >>= st == 32 ? 2 : 1) sum[e] += __shfl_xor(sum[e], st, 64);
            if (r == 0 && g < 2)
#pragma unroll
                for (int e = 0; e < 4; ++e) wave_sum[wave][4 * g + e] = sum[e];
            __syncthreads();
            double v = 0.0;
            for (int w = 0; w < S::WAVES; ++w) v += wave_sum[w][threadIdx.x & 7];
            return v;
        };
        double v = totals();
        if (__any(isnan(v))) {                              // (the same in every wave)
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] = 0.0;
            apart();
            v = totals();
        }
        if (threadIdx.x < 8) A.sums[(size_t)blockIdx.x * 8 + threadIdx.x] = v;
    } else if constexpr (FOLD) {
        if (__syncthreads_or(nan)) apart();
    }
}
#undef INLINE

// one workgroup per CU, or one per tile: multiples of 8
template <int CIN, int COUT>
static int conv_grid(const int n[3])
{
    const int ntiles = (n[0] / CT_X) * (n[1] / CT_Y) * (n[2] / ConvShape<CIN, COUT>::TZ);
    return ntiles < CONV_WGS ? ntiles : CONV_WGS;
}
int closure_sum_blocks(const int n[3]) { return conv_grid<32, 8>(n); }

template <int CIN, int COUT, int EPI>
static hipError_t conv_launch(const ConvArgs& A, hipStream_t s)
{
    using S = ConvShape<CIN, COUT>;
    const dim3 grid((unsigned)conv_grid<CIN, COUT>(A.n)), block(S::THREADS);
    const unsigned long long pieces = (unsigned long long)S::PARTS * A.n[0] * A.n[1] * A.n[2];
    // offsets in 32 bits up to 2^30 cells of 32 channels (64 GiB); past that
    // only the single-layer calls get (a closure's buffers take 400 GiB there)
    if (pieces < 1ull << 32) hipLaunchKernelGGL((conv3d_kernel<CIN, COUT, EPI, unsigned>), grid, block, 0, s, A);
    else if constexpr (EPI == EPI_BIAS_F32 || EPI == EPI_F32)
        hipLaunchKernelGGL((conv3d_kernel<CIN, COUT, EPI, unsigned long long>), grid, block, 0, s, A);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

template <int CIN, int COUT>
static hipError_t conv_dispatch_epi(const ConvArgs& A, int epi, hipStream_t s)
{
    switch (epi) {
    case EPI_BIAS_RELU:
        if constexpr (COUT == 32) return conv_launch<CIN, COUT, EPI_BIAS_RELU>(A, s);
        return hipErrorInvalidValue;
    case EPI_BIAS_F32: return conv_launch<CIN, COUT, EPI_BIAS_F32>(A, s);
    case EPI_MASK:
        if constexpr (COUT == 32) return conv_launch<CIN, COUT, EPI_MASK>(A, s);
        return hipErrorInvalidValue;
    case EPI_F32: return conv_launch<CIN, COUT, EPI_F32>(A, s);
    case EPI_CLOSURE:
        if constexpr (CIN == 32 && COUT == 8) return conv_launch<CIN, COUT, EPI_CLOSURE>(A, s);
        return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_conv3d(const ConvArgs& A, int cin, int cout, int epi, hipStream_t s)
{
    if (cin == 8 && cout == 32) return conv_dispatch_epi<8, 32>(A, epi, s);
    if (cin == 32 && cout == 32) return conv_dispatch_epi<32, 32>(A, epi, s);
    if (cin == 32 && cout == 8) return conv_dispatch_epi<32, 8>(A, epi, s);
    if (cin == 8 && cout == 8) return conv_dispatch_epi<8, 8>(A, epi, s);
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// reductions over workgroups
// ---------------------------------------------------------------------------

// Sums of NV FP64 values per thread over the 256 threads of a workgroup, to
// every thread: a fixed tree over the lanes, then the four waves in order.
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV])
{
    __shared__ double sh[NV][4];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
#pragma unroll
        for (int st = 32; st > 0; st >>= 1) v[q] += __shfl_xor(v[q], st, 64);
        if ((threadIdx.x & 63) == 0) sh[q][threadIdx.x >> 6] = v[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = ((sh[q][0] + sh[q][1]) + sh[q][2]) + sh[q][3];
}

// Totals of the nblk workgroups' sums partial[b * stride + first + q] of the
// launch before, by every workgroup for itself: a launch of one workgroup for
// them took 5 to 6 us, as long as the pass that needs them at 64^3.
template <int NV>
__device__ __forceinline__ void block_totals(const double* __restrict__ partial, int nblk, int stride, int first,
                                             double (&total)[NV])
{
#pragma unroll
    for (int q = 0; q < NV; ++q) total[q] = 0.0;
    for (int b = threadIdx.x; b < nblk; b += 256)
#pragma unroll
        for (int q = 0; q < NV; ++q) total[q] += partial[(size_t)b * stride + first + q];
    block_sum(total);
}

// ---------------------------------------------------------------------------
// wgrad
// ---------------------------------------------------------------------------

// dW[o][ci][co] = sum_c x[c + d(o)][ci] dy[c][co] as MFMA products with M =
// co, N = ci, K = cells.  Both operands are staged as they lie in memory,
// channel-last; the fragments, whose lanes want 8 consecutive cells of one
// channel, come from ds_read_b64_tr_b16: in each group of 16 lanes, lane i
// gives the address of 4 channels (4 (i % 4) ..) of cell i / 4 and receives
// channel i of the 4 cells.  An offset d(o) is then only another address, with
// no shifting and no channel-major copy of any activation (the form before
// read such copies, which the producing kernels wrote 2 bytes at a time).
//
// Tile: 32 (x) x 4 (y) x 2 (z) cells, x with a one-cell halo.  Six waves: wave
// w has the offsets with dz = w / 2 - 1 and half of the blocks (32 -> 32: 16
// of the ci; 8 -> 32: 16 of the co; 32 -> 8: 16 of the ci).  A row of x is
// read once per dx and multiplies the rows y - dy of dy of all three dy, kept
// in registers: 52 reads of 512 bytes feed 72 products per plane.  Two
// workgroups fit on a CU, so that one's products cover the other's staging.
// Where one side has 8 channels the 16 rows (columns) of a block hold two
// offsets: for 8 input channels columns 8 .. 15 read the next cell (dx + 1),
// for 8 output channels rows 8 .. 15 read the cell before of dy, which turns
// dx into dx + 1.  Two blocks then make the three dx.
//
// Persistent over tiles (XCD k takes the k-th eighth, so that halos shared by
// neighbouring tiles meet in its L2); each workgroup writes its partial sums
// of dW and, in FP64, of the bias gradient, wgrad_reduce_kernel adds them in a
// fixed order.
constexpr int WT_X = 32, WT_Y = 4, WT_Z = 2;
constexpr int WL_X = WT_X + 2, WL_Y = WT_Y + 2, WL_Z = WT_Z + 2;

template <int CI, int CO>
struct WgradShape {
    static constexpr bool FM = CO == 8 && CI == 32;        // rows hold two offsets
    static constexpr bool FN = CI == 8;                    // columns do
    static constexpr int WAVES = CI == 8 && CO == 8 ? 3 : 6;
    static constexpr int HALVES = WAVES / 3;
    static constexpr int ND = FM || FN ? 2 : 3;            // x blocks (dx) per row of x and wave
    static constexpr int MB = CI == 32 && CO == 32 ? 2 : 1;     // dy blocks per row of dy and wave
    static constexpr int DX = FM ? WT_X + 1 : WT_X;        // dy cells per row (FM: one before)
    static constexpr int XS = WL_Z * WL_Y * WL_X * CI, DS = WT_Z * WT_Y * DX * CO;
};

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s4;

// 8 cells of a channel: two transposing reads, the second 4 cells on
__device__ __forceinline__ bf16x8 read_cells(const uint16_t* p, int step4)
{
    typedef __attribute__((address_space(3))) s4* lds4;
    const s4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)p);
    const s4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(p + step4));
    typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s8;
    return __builtin_bit_cast(bf16x8, s8{ a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3] });
}

template <int CI, int CO>
__global__ void __launch_bounds__((64 * WgradShape<CI, CO>::WAVES), 3) conv3d_wgrad_kernel(WgradArgs A)
{
    using S = WgradShape<CI, CO>;
    constexpr int NT = 64 * S::WAVES, ND = S::ND, MB = S::MB;
    // dy behind x: the last folded columns read one cell past x's last row
    __shared__ __align__(16) uint16_t smem[S::XS + S::DS];
    uint16_t* const xs = smem;
    uint16_t* const ds = smem + S::XS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane >> 4, i = lane & 15;
    const int dz = wave / S::HALVES, half = wave % S::HALVES;
    const int nx = A.n[0], ny = A.n[1], nz = A.n[2];
    const int tx = nx / WT_X, ty = ny / WT_Y, per = (tx * ty * (nz / WT_Z)) >> 3;

    // lane bases: cell 8 g + i / 4, channels 4 (i % 4) .. of the wave's block;
    // folded: channels 4 (i % 2) .. of this cell or, for i % 4 >= 2, of the other
    const int c0 = 8 * g + (i >> 2);
    const uint16_t* const xb = xs + dz * (WL_Y * WL_X * CI) +
                               (S::FN ? (c0 + ((i >> 1) & 1)) * CI + 4 * (i & 1) : c0 * CI + 16 * half + 4 * (i & 3));
    const uint16_t* const db = ds + (S::FM    ? (c0 + 1 - ((i >> 1) & 1)) * CO + 4 * (i & 1)
                                     : CO == 8 ? c0 * CO + 4 * (i & 1)
                                               : c0 * CO + (S::FN ? 16 * half : 0) + 4 * (i & 3));

    f4 acc[3][ND][MB];                                      // [dy][block of dx][m]
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int d = 0; d < ND; ++d)
#pragma unroll
            for (int m = 0; m < MB; ++m) acc[a][d][m] = f4{ 0.f, 0.f, 0.f, 0.f };
    // bias: thread t < BT sums 8 channels of the cells t / (CO / 8) + BT / (CO / 8) j
    constexpr int BT = NT < 256 ? 128 : 256, BQ = CO / 8, BSTEP = BT / BQ;
    double bias[8] = { 0, 0, 0, 0, 0, 0, 0, 0 };

    for (int t = (blockIdx.x & 7) * per + (blockIdx.x >> 3); t < ((blockIdx.x & 7) + 1) * per; t += gridDim.x >> 3) {
        const int x0 = (t % tx) * WT_X, y0 = ((t / tx) % ty) * WT_Y, z0 = (t / (tx * ty)) * WT_Z;
        // two batches of loads for 32 -> 32 channels: 12 in flight would spill
        // at 3 waves per SIMD
        constexpr int XI = S::XS / 8, ITEMS = (S::XS + S::DS) / 8, FILL = (ITEMS + NT - 1) / NT;
        constexpr int FB = FILL > 8 ? (FILL + 1) / 2 : FILL;
        int tid = threadIdx.x;
        // opaque with 32 -> 32 channels, where the places of all pieces, kept
        // in registers over the loop, would spill
        if constexpr (CI * CO > 256) asm volatile("" : "+v"(tid));
        auto item = [&](int f) { return min(tid + NT * f, ITEMS - 1); };     // past the end: the last piece again
#pragma unroll
        for (int f0 = 0; f0 < FILL; f0 += FB) {
            uint4 fv[FB];
#pragma unroll
            for (int f = 0; f < FB; ++f) {
                const int it = item(f0 + f);
                const bool isx = it < XI;
                const int d = isx ? it : it - XI;
                const int q = isx ? d % (CI / 8) : d % (CO / 8), c = isx ? d / (CI / 8) : d / (CO / 8);
                const int cx = isx ? c % WL_X - 1 : c % S::DX - (S::FM ? 1 : 0), row = isx ? c / WL_X : c / S::DX;
                const int cy = isx ? row % WL_Y - 1 : row % WT_Y, cz = isx ? row / WL_Y - 1 : row / WT_Y;
                const unsigned src = (unsigned)wrap1(x0 + cx, nx) +
                                     (unsigned)nx * ((unsigned)wrap1(y0 + cy, ny) + (unsigned)ny * (unsigned)wrap1(z0 + cz, nz));
                fv[f] = ld16(isx ? A.x + (size_t)src * CI + 8 * q : A.dy + (size_t)src * CO + 8 * q);
            }
            if (f0 == 0) __syncthreads();                  // the previous tile's reads are done
#pragma unroll
            for (int f = 0; f < FB; ++f) *reinterpret_cast<uint4*>(smem + 8 * item(f0 + f)) = fv[f];
        }
        __syncthreads();
        if (threadIdx.x < BT) {
            float part[8] = { 0, 0, 0, 0, 0, 0, 0, 0 };
#pragma unroll
            for (int j = 0; j < 256 / BSTEP; ++j) {
                const int c = threadIdx.x / BQ + BSTEP * j;
                const uint4 v = *reinterpret_cast<const uint4*>(ds + (c + (S::FM ? c / WT_X + 1 : 0)) * CO + 8 * (threadIdx.x % BQ));
                const uint32_t w[4] = { v.x, v.y, v.z, v.w };
#pragma unroll
                for (int e = 0; e < 8; ++e) part[e] += bf2f((uint16_t)(w[e >> 1] >> (16 * (e & 1))));
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) bias[e] += (double)part[e];
        }
#pragma unroll 1
        for (int kz = 0; kz < WT_Z; ++kz) {
            bf16x8 a[WT_Y][MB];
#pragma unroll
            for (int ky = 0; ky < WT_Y; ++ky)
#pragma unroll
                for (int m = 0; m < MB; ++m) a[ky][m] = read_cells(db + (kz * WT_Y + ky) * (S::DX * CO) + 16 * m, 4 * CO);
#pragma unroll
            for (int row = 0; row < WL_Y; ++row) {
                bf16x8 b[ND];
#pragma unroll
                for (int d = 0; d < ND; ++d)
                    b[d] = read_cells(xb + ((kz * WL_Y + row) * WL_X + (ND == 2 ? 2 * d : d)) * CI, 4 * CI);
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                    const int ky = row - dy;
                    if (ky < 0 || ky >= WT_Y) continue;
#pragma unroll
                    for (int d = 0; d < ND; ++d)
#pragma unroll
                        for (int m = 0; m < MB; ++m)
                            acc[dy][d][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ky][m], b[d], acc[dy][d][m], 0, 0, 0);
                }
            }
        }
    }
    // D of a block: lane holds rows 4 g + e (e = 0..3), column i
    float* const out = A.partial + (size_t)blockIdx.x * 27 * CI * CO;
#pragma unroll
    for (int dy = 0; dy < 3; ++dy)
#pragma unroll
        for (int d = 0; d < ND; ++d)
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                const int row = 4 * g;
                const int co = S::FM || CO == 8 ? row & 7 : (S::FN ? 16 * half : 16 * m) + row;
                const int ci = S::FN ? i & 7 : 16 * half + i;
                const int dx = ND == 2 ? 2 * d + (S::FN ? i >> 3 : row >> 3) : d;
                if (dx > 2 || (CO == 8 && !S::FM && row >= 8)) continue;
                const int o = dz * 9 + dy * 3 + dx;
                *reinterpret_cast<f4*>(out + ((size_t)o * CI + ci) * CO + co) = acc[dy][d][m];
            }
    // bias: threads of a chunk of channels added in order
    __syncthreads();
    double* const sh = reinterpret_cast<double*>(smem);
    if (threadIdx.x < BT)
#pragma unroll
        for (int e = 0; e < 8; ++e) sh[e * BT + threadIdx.x] = bias[e];
    __syncthreads();
    if (threadIdx.x < CO) {
        double v = 0.0;
        for (int j = threadIdx.x >> 3; j < BT; j += BQ) v += sh[(threadIdx.x & 7) * BT + j];
        A.bias_partial[(size_t)blockIdx.x * CO + threadIdx.x] = v;
    }
}

// grads of up to 3 layers from their workgroups' partial sums, in workgroup
// order: a block of 256 threads takes 64 consecutive weights, thread group j
// the j-th quarter of the workgroups (8 running sums each), then the quarters
// in order; the blocks past the weights take the biases, the last one the loss
struct WgradReduce {
    WgradLayer layer[3];
    int nlayer, nwg;
    const double* loss_partial;                             // LOSS_SUMS per workgroup, or null
    int nloss;
    double loss_scale;
    double* loss;
};
constexpr int WR_GROUPS = 4, WR_SUMS = 8;
__global__ void __launch_bounds__(256) wgrad_reduce_kernel(WgradReduce R)
{
    int b = blockIdx.x, l = 0;
    if (R.loss_partial && blockIdx.x == gridDim.x - 1) {
        double total[1];
        block_totals(R.loss_partial, R.nloss, LOSS_SUMS, 0, total);
        if (threadIdx.x == 0) *R.loss = total[0] * R.loss_scale;
        return;
    }
    while (l < R.nlayer && b >= (R.layer[l].count + 63) / 64) b -= (R.layer[l++].count + 63) / 64;
    if (l == R.nlayer) {                                   // biases: a wave per channel
        int c = 4 * b + (threadIdx.x >> 6);
        for (l = 0; l < R.nlayer && c >= R.layer[l].cout; ++l) c -= R.layer[l].cout;
        if (l == R.nlayer) return;
        double v = 0.0;
        for (int w = threadIdx.x & 63; w < R.nwg; w += 64) v += R.layer[l].bias_partial[(size_t)w * R.layer[l].cout + c];
#pragma unroll
        for (int st = 32; st > 0; st >>= 1) v += __shfl_xor(v, st, 64);
        if ((threadIdx.x & 63) == 0) R.layer[l].dbias[c] = (float)v;
        return;
    }
    const WgradLayer& L = R.layer[l];
    const int e = threadIdx.x & 63, j = threadIdx.x >> 6;
    const int k = b * 64 + e;                              // counts are multiples of 64
    const int per = (R.nwg + WR_GROUPS - 1) / WR_GROUPS;
    const int w0 = j * per, w1 = min(R.nwg, w0 + per);
    float acc[WR_SUMS] = {};
    int w = w0;
    for (; w + WR_SUMS <= w1; w += WR_SUMS)
#pragma unroll
        for (int q = 0; q < WR_SUMS; ++q) acc[q] += L.partial[(size_t)(w + q) * L.count + k];
    for (int q = 0; w < w1; ++w, ++q) acc[q] += L.partial[(size_t)w * L.count + k];
    __shared__ float sh[WR_GROUPS][64];
    sh[j][e] = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
    __syncthreads();
    if (j == 0) L.dw[k] = (sh[0][e] + sh[1][e]) + (sh[2][e] + sh[3][e]);
}

// Workgroups of a wgrad launch, a multiple of 8: two per CU; one where that
// leaves them fewer than 8 tiles each, as every workgroup's 110 KiB of partial
// sums are written and read again.
int wgrad_blocks(const int n[3])
{
    const int ntiles = (n[0] / WT_X) * (n[1] / WT_Y) * (n[2] / WT_Z);
    const int most = ntiles >= 8 * WGRAD_MAX_WG ? WGRAD_MAX_WG : WGRAD_MAX_WG / 2;
    return ntiles < most ? ntiles : most;
}

hipError_t launch_conv3d_wgrad(const WgradArgs& A, int cin, int cout, hipStream_t s)
{
    const int nwg = wgrad_blocks(A.n);
    if (cin == 8 && cout == 32)
        hipLaunchKernelGGL((conv3d_wgrad_kernel<8, 32>), dim3(nwg), dim3(64 * WgradShape<8, 32>::WAVES), 0, s, A);
    else if (cin == 32 && cout == 32)
        hipLaunchKernelGGL((conv3d_wgrad_kernel<32, 32>), dim3(nwg), dim3(64 * WgradShape<32, 32>::WAVES), 0, s, A);
    else if (cin == 32 && cout == 8)
        hipLaunchKernelGGL((conv3d_wgrad_kernel<32, 8>), dim3(nwg), dim3(64 * WgradShape<32, 8>::WAVES), 0, s, A);
    else if (cin == 8 && cout == 8)
        hipLaunchKernelGGL((conv3d_wgrad_kernel<8, 8>), dim3(nwg), dim3(64 * WgradShape<8, 8>::WAVES), 0, s, A);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_wgrad_reduce(const WgradLayer* layers, int nlayer, int nwg, const double* loss_partial, size_t N,
                               double* loss, hipStream_t s)
{
    WgradReduce R;
    int blocks = loss_partial ? 1 : 0;
    R.loss_partial = loss_partial;
    R.nloss = loss_partial ? loss_blocks(N) : 0;
    R.loss_scale = 1.0 / (8.0 * (double)N);
    R.loss = loss;
    R.nlayer = nlayer;
    R.nwg = nwg;
    for (int l = 0; l < nlayer; ++l) {
        R.layer[l] = layers[l];
        blocks += (layers[l].count + 63) / 64 + layers[l].cout / 4;     // 64 weights or 4 biases each
    }
    hipLaunchKernelGGL(wgrad_reduce_kernel, dim3(blocks), dim3(256), 0, s, R);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// conversions
// ---------------------------------------------------------------------------

// bf16 [c][cell] -> [cell][c] (c = 8 or 32; the single-layer entry point takes
// channel-major operands): a workgroup takes 64 cells, through LDS
template <int C>
__global__ void __launch_bounds__(256) channel_last_kernel(const uint16_t* __restrict__ src, size_t N, uint16_t* __restrict__ dst)
{
    __shared__ uint16_t sh[64][C + 2];
    const size_t c0 = (size_t)blockIdx.x * 64;
    for (int t = threadIdx.x; t < 64 * C; t += 256) sh[t & 63][t >> 6] = src[(size_t)(t >> 6) * N + c0 + (t & 63)];
    __syncthreads();
    for (int t = threadIdx.x; t < 64 * C; t += 256) dst[c0 * C + t] = sh[t / C][t % C];
}

hipError_t launch_channel_last(const uint16_t* src, size_t N, int c, uint16_t* dst, hipStream_t s)
{
    if (c == 8) hipLaunchKernelGGL(channel_last_kernel<8>, dim3((unsigned)(N / 64)), dim3(256), 0, s, src, N, dst);
    else if (c == 32) hipLaunchKernelGGL(channel_last_kernel<32>, dim3((unsigned)(N / 64)), dim3(256), 0, s, src, N, dst);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// closure elementwise and reduction kernels
// ---------------------------------------------------------------------------
// States are FP32 field-major u[f][cell]; the network sees x[cell][8] =
// (u - mean) / std in bf16.

// A state's fields: the fluid fields from one base, the faces from another
// (the two may sit in different buffers of a solver).
__device__ __forceinline__ const float* field(const ClosureState& u, int f, size_t N)
{
    return (f < 5 ? u.fluid : u.faces) + (size_t)f * N;
}

__global__ void normalize_kernel(ClosureState u, size_t N, ClosureScales sc, uint16_t* __restrict__ x)
{
    for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < N; c += (size_t)gridDim.x * blockDim.x) {
        float b[8];
#pragma unroll
        for (int f = 0; f < 8; ++f) b[f] = (field(u, f, N)[c] - sc.in_mean[f]) / sc.in_std[f];
        *reinterpret_cast<uint4*>(x + c * 8) =
            make_uint4(f2bf2(b[0], b[1]), f2bf2(b[2], b[3]), f2bf2(b[4], b[5]), f2bf2(b[6], b[7]));
    }
}

hipError_t launch_normalize(const ClosureState& u, size_t N, const ClosureScales& sc, uint16_t* x, hipStream_t s)
{
    hipLaunchKernelGGL(normalize_kernel, dim3(2048), dim3(256), 0, s, u, N, sc, x);
    return hipGetLastError();
}

// The passes over cells between the convolutions are bound by memory, so each
// value is read as few times as its producers and readers allow: the gate and
// the network's input come from one read of the state, the gate is applied
// and the channel sums taken where the last layer's outputs are registers,
// and the loss is taken where the correction is.  128^3, gated forward:
// normalise + gate + scale + sums + projection + copy of the result 151 us ->
// 77 us; 96 x 64 x 64 forward and backward, from 15 launches to 7.
//
// delta[f][c] = s_f (o[c][f] - mean_f) (f < 5); delta_b = curl of A = s (o5,
// o6, o7), the means from the convolution's channel sums.  TRAIN: instead of
// storing delta, the loss against target in the same pass: r = (delta -
// target) / t_f, g = 2 r / t_f / (8 N), and per workgroup the sums of r^2 and
// of the five fluid g (LOSS_SUMS values).  clear (may be null): set to 0.
struct LossScales {
    double g[8];        // 2 / t_f / (8 N): FP64 divisions, once on the host
};
template <bool TRAIN>
__global__ void __launch_bounds__(256) project_kernel(const float* __restrict__ o, const double* __restrict__ sums,
                                                      int nsums, int nx, int ny, int nz, ClosureScales sc,
                                                      float* __restrict__ delta, const float* __restrict__ target,
                                                      LossScales ls, double* __restrict__ partial, int* clear)
{
    const size_t N = (size_t)nx * ny * nz;
    double mean[5];
    block_totals(sums, nsums, 8, 0, mean);
#pragma unroll
    for (int f = 0; f < 5; ++f) mean[f] *= 1.0 / (double)N;
    if (clear && blockIdx.x == 0 && threadIdx.x == 0) *clear = 0;
    double acc[LOSS_SUMS] = { 0, 0, 0, 0, 0, 0 };
    for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < N; c += (size_t)gridDim.x * blockDim.x) {
        int i, j, k;
        cell_ijk((unsigned)c, nx, ny, i, j, k);
        const float4 lo = *reinterpret_cast<const float4*>(o + c * 8), hi = *reinterpret_cast<const float4*>(o + c * 8 + 4);
        const float oc[8] = { lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w };
        float d[8];
#pragma unroll
        for (int f = 0; f < 5; ++f) d[f] = sc.out_scale[f] * (float)((double)oc[f] - mean[f]);
        const size_t cxp = (size_t)wrap1(i + 1, nx) + (size_t)nx * (j + (size_t)ny * k);
        const size_t cyp = (size_t)i + (size_t)nx * (wrap1(j + 1, ny) + (size_t)ny * k);
        const size_t czp = (size_t)i + (size_t)nx * (j + (size_t)ny * wrap1(k + 1, nz));
        const float s5 = sc.out_scale[5], s6 = sc.out_scale[6], s7 = sc.out_scale[7];
        const float ax = s5 * oc[5], ay = s6 * oc[6], az = s7 * oc[7];
        d[5] = (s7 * o[cyp * 8 + 7] - az) - (s6 * o[czp * 8 + 6] - ay);
        d[6] = (s5 * o[czp * 8 + 5] - ax) - (s7 * o[cxp * 8 + 7] - az);
        d[7] = (s6 * o[cxp * 8 + 6] - ay) - (s5 * o[cyp * 8 + 5] - ax);
#pragma unroll
        for (int f = 0; f < 8; ++f) {
            if constexpr (TRAIN) {
                const float ts = sc.target_scale[f];
                const float r = (d[f] - target[(size_t)f * N + c]) / ts;
                const float g = (float)((double)r * ls.g[f]);
                acc[0] += (double)r * (double)r;
                if (f < 5) acc[1 + f] += (double)g;
                delta[(size_t)f * N + c] = g;
            } else {
                delta[(size_t)f * N + c] = d[f];
            }
        }
    }
    if constexpr (TRAIN) {
        block_sum(acc);
        if (threadIdx.x == 0)
#pragma unroll
            for (int q = 0; q < LOSS_SUMS; ++q) partial[(size_t)blockIdx.x * LOSS_SUMS + q] = acc[q];
    }
}

// one cell per thread up to LOSS_BLOCKS workgroups
static unsigned cell_blocks(size_t N)
{
    const size_t b = (N + 255) / 256;
    return (unsigned)(b < LOSS_BLOCKS ? b : LOSS_BLOCKS);
}
int loss_blocks(size_t N) { return (int)cell_blocks(N); }

hipError_t launch_project(const float* o, const double* sums, int nsums, const int n[3], const ClosureScales& sc,
                          float* delta, int* clear, hipStream_t s)
{
    hipLaunchKernelGGL(project_kernel<false>, dim3(cell_blocks((size_t)n[0] * n[1] * n[2])), dim3(256), 0, s, o, sums,
                       nsums, n[0], n[1], n[2], sc, delta, nullptr, LossScales{}, nullptr, clear);
    return hipGetLastError();
}

hipError_t launch_project_loss(const float* o, const double* sums, int nsums, const int n[3], const ClosureScales& sc,
                               const float* target, float* g, double* partial, hipStream_t s)
{
    const size_t N = (size_t)n[0] * n[1] * n[2];
    LossScales ls;
    for (int f = 0; f < 8; ++f) ls.g[f] = 2.0 / (double)sc.target_scale[f] / (8.0 * (double)N);
    hipLaunchKernelGGL(project_kernel<true>, dim3(cell_blocks(N)), dim3(256), 0, s, o, sums, nsums, n[0], n[1], n[2],
                       sc, g, target, ls, partial, nullptr);
    return hipGetLastError();
}

// adjoint of the projection, g[f][c] -> go[c][8], times the gate (gate may be
// null) and rounded to bf16: the output gradient as dgrad and wgrad read it.
// partial: the workgroups' sums of project_kernel<true>.
__global__ void __launch_bounds__(256) project_T_kernel(const float* __restrict__ g, const double* __restrict__ partial,
                                                        int npartial, const float* __restrict__ gate, int nx, int ny,
                                                        int nz, ClosureScales sc, uint16_t* __restrict__ go)
{
    const size_t N = (size_t)nx * ny * nz;
    double gmean[5];
    block_totals(partial, npartial, LOSS_SUMS, 1, gmean);
#pragma unroll
    for (int f = 0; f < 5; ++f) gmean[f] *= 1.0 / (double)N;
    for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < N; c += (size_t)gridDim.x * blockDim.x) {
        int i, j, k;
        cell_ijk((unsigned)c, nx, ny, i, j, k);
        float v[8];
#pragma unroll
        for (int f = 0; f < 5; ++f) v[f] = sc.out_scale[f] * (float)((double)g[(size_t)f * N + c] - gmean[f]);
        const size_t cxm = (size_t)wrap1(i - 1, nx) + (size_t)nx * (j + (size_t)ny * k);
        const size_t cym = (size_t)i + (size_t)nx * (wrap1(j - 1, ny) + (size_t)ny * k);
        const size_t czm = (size_t)i + (size_t)nx * (j + (size_t)ny * wrap1(k - 1, nz));
        const float* gx = g + 5 * N;
        const float* gy = g + 6 * N;
        const float* gz = g + 7 * N;
        v[7] = sc.out_scale[7] * ((gx[cym] - gx[c]) - (gy[cxm] - gy[c]));
        v[6] = sc.out_scale[6] * ((gz[cxm] - gz[c]) - (gx[czm] - gx[c]));
        v[5] = sc.out_scale[5] * ((gy[czm] - gy[c]) - (gz[cym] - gz[c]));
        if (gate) {
            const float s = gate[c];
#pragma unroll
            for (int f = 0; f < 8; ++f) v[f] *= s;
        }
        *reinterpret_cast<uint4*>(go + c * 8) =
            make_uint4(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]), f2bf2(v[4], v[5]), f2bf2(v[6], v[7]));
    }
}

hipError_t launch_project_T(const float* g, const double* partial, const float* gate, const int n[3],
                            const ClosureScales& sc, uint16_t* go, hipStream_t s)
{
    const size_t N = (size_t)n[0] * n[1] * n[2];
    hipLaunchKernelGGL(project_T_kernel, dim3(cell_blocks(N)), dim3(256), 0, s, g, partial, loss_blocks(N), gate, n[0],
                       n[1], n[2], sc, go);
    return hipGetLastError();
}

// Guard of the corrected state u + theta delta for theta = 2^-k, k = 0..3:
// bit k of *bad is raised if some cell has rho <= 0, p < 0 or a non-finite
// value at that theta (pressure from the cell-centred field, the mean of
// the two faces; tested without a division as 2 rho (e - |B|^2/2) >= |m|^2).
__global__ void __launch_bounds__(256) guard_levels_kernel(ClosureState u, const float* __restrict__ delta, int nx,
                                                          int ny, int nz, int* bad)
{
    // 4 consecutive x cells per thread (nx is a multiple of 4)
    const unsigned N = (unsigned)nx * ny * nz, N4 = N / 4;
    int b = 0;
    for (unsigned t = blockIdx.x * blockDim.x + threadIdx.x; t < N4; t += gridDim.x * blockDim.x) {
        const unsigned c = 4 * t;
        int i, j, k;
        cell_ijk(c, nx, ny, i, j, k);
        const unsigned xp = c - i + wrap1(i + 4, nx);
        const unsigned cyp = (unsigned)i + (unsigned)nx * ((unsigned)wrap1(j + 1, ny) + (unsigned)ny * k);
        const unsigned czp = (unsigned)i + (unsigned)nx * ((unsigned)j + (unsigned)ny * wrap1(k + 1, nz));
        float u0[8][4], d0[8][4], u1[3][4], d1[3][4];
        for (int f = 0; f < 8; ++f) {
            const float4 a4 = *reinterpret_cast<const float4*>(field(u, f, N) + c);
            const float4 b4 = *reinterpret_cast<const float4*>(delta + (size_t)f * N + c);
            u0[f][0] = a4.x; u0[f][1] = a4.y; u0[f][2] = a4.z; u0[f][3] = a4.w;
            d0[f][0] = b4.x; d0[f][1] = b4.y; d0[f][2] = b4.z; d0[f][3] = b4.w;
        }
        // upper faces: b_x of the next cell along x, b_y / b_z of the next row / plane
        for (int q = 0; q < 3; ++q) { u1[0][q] = u0[5][q + 1]; d1[0][q] = d0[5][q + 1]; }
        u1[0][3] = field(u, 5, N)[xp];
        d1[0][3] = delta[(size_t)5 * N + xp];
        {
            const float4 a4 = *reinterpret_cast<const float4*>(field(u, 6, N) + cyp);
            const float4 b4 = *reinterpret_cast<const float4*>(delta + (size_t)6 * N + cyp);
            const float4 c4 = *reinterpret_cast<const float4*>(field(u, 7, N) + czp);
            const float4 e4 = *reinterpret_cast<const float4*>(delta + (size_t)7 * N + czp);
            u1[1][0] = a4.x; u1[1][1] = a4.y; u1[1][2] = a4.z; u1[1][3] = a4.w;
            d1[1][0] = b4.x; d1[1][1] = b4.y; d1[1][2] = b4.z; d1[1][3] = b4.w;
            u1[2][0] = c4.x; u1[2][1] = c4.y; u1[2][2] = c4.z; u1[2][3] = c4.w;
            d1[2][0] = e4.x; d1[2][1] = e4.y; d1[2][2] = e4.z; d1[2][3] = e4.w;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int lev = 0; lev < GUARD_LEVELS; ++lev) {
                const float th = ldexpf(1.0f, -lev);
                float v[8];
                bool ok = true;
                for (int f = 0; f < 8; ++f) {
                    v[f] = u0[f][q] + th * d0[f][q];
                    ok = ok && isfinite(v[f]);
                }
                float b2 = 0.0f;
                for (int a = 0; a < 3; ++a) {
                    const float bc = 0.5f * (v[5 + a] + (u1[a][q] + th * d1[a][q]));
                    b2 += bc * bc;
                }
                // p >= 0 with rho > 0  <=>  2 rho (e - |B|^2 / 2) >= |m|^2 (gamma > 1)
                const float lhs = 2.0f * v[0] * (v[4] - 0.5f * b2);
                const float m2 = v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
                ok = ok && v[0] > 0.0f && lhs >= m2;
                if (!ok) b |= 1 << lev;
            }
    }
    // one atomic per wave: OR of the level bits over its lanes
    int wb = 0;
#pragma unroll
    for (int lev = 0; lev < GUARD_LEVELS; ++lev)
        if (__ballot((b >> lev) & 1)) wb |= 1 << lev;
    if ((threadIdx.x & 63) == 0 && wb) atomicOr(bad, wb);
}

hipError_t launch_guard_levels(const ClosureState& u, const float* delta, const int n[3], float gamma, int* bad,
                               hipStream_t s)
{
    (void)gamma;                      // the sign of p does not depend on gamma > 1
    hipLaunchKernelGGL(guard_levels_kernel, dim3(2048), dim3(256), 0, s, u, delta, n[0], n[1], n[2], bad);
    return hipGetLastError();
}

// out = u + theta delta with the largest theta = 2^-k whose guard bit is
// clear; none clear: out = u (the plain step).  out may hold part of u.
// counts[0] counts dropped corrections, counts[1] reduced ones (theta < 1).
// 4 values per thread: a field is a multiple of 4 long.
__global__ void __launch_bounds__(256) apply_level_kernel(ClosureState u, const float* __restrict__ delta, size_t N,
                                                          const int* bad, int* counts, float* out)
{
    const int mask = *bad;
    int lev = 0;
    while (lev < GUARD_LEVELS && (mask >> lev) & 1) ++lev;
    if (blockIdx.x == 0 && threadIdx.x == 0 && counts) {
        if (lev == GUARD_LEVELS) counts[0] += 1;
        else if (lev > 0) counts[1] += 1;
    }
    const float th = ldexpf(1.0f, -lev);
    for (size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x; t < 2 * N; t += (size_t)gridDim.x * blockDim.x) {
        const float* const src = 4 * t < 5 * N ? u.fluid : u.faces;
        if (lev == GUARD_LEVELS && src == out) continue;
        float4 v = reinterpret_cast<const float4*>(src)[t];
        if (lev < GUARD_LEVELS) {
            const float4 d = reinterpret_cast<const float4*>(delta)[t];
            v.x = v.x + th * d.x; v.y = v.y + th * d.y; v.z = v.z + th * d.z; v.w = v.w + th * d.w;
        }
        reinterpret_cast<float4*>(out)[t] = v;
    }
}

hipError_t launch_apply_level(const ClosureState& u, const float* delta, size_t N, const int* bad, int* counts,
                              float* out, hipStream_t s)
{
    hipLaunchKernelGGL(apply_level_kernel, dim3(2048), dim3(256), 0, s, u, delta, N, bad, counts, out);
    return hipGetLastError();
}

// Adam (Kingma & Ba) on FP32 master parameters
__global__ void adam_kernel(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, int n, float lr, float b1, float b2, float eps, float c1, float c2)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

hipError_t launch_adam(float* p, const float* g, float* m, float* v, int n, float lr, float b1, float b2, float eps,
                       int step, hipStream_t s)
{
    const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    hipLaunchKernelGGL(adam_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, g, m, v, n, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

// target = u_ref - u_plain, elementwise over 8N values
__global__ void residual_kernel(const float* __restrict__ ref, const float* __restrict__ plain, size_t n,
                                float* __restrict__ out)
{
    for (size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x)
        out[t] = ref[t] - plain[t];
}

hipError_t launch_residual(const float* ref, const float* plain, size_t n, float* out, hipStream_t s)
{
    hipLaunchKernelGGL(residual_kernel, dim3(2048), dim3(256), 0, s, ref, plain, n, out);
    return hipGetLastError();
}

// Per-field sums of a field-major pair (u, t), blockIdx.y = field:
// partial[(b * 8 + f) * 5 + q], q = sum u, sum u^2, sum |u|, sum |t|, and
// sum of the roughness r = sum over axes |u(c+a) - 2 u(c) + u(c-a)|
__global__ void __launch_bounds__(256) stats_partial_kernel(const float* __restrict__ u,
                                                            const float* __restrict__ t, int nx, int ny, int nz,
                                                            double* __restrict__ partial)
{
    const size_t N = (size_t)nx * ny * nz;
    const int f = blockIdx.y;
    const float* uf = u + (size_t)f * N;
    const float* tf = t + (size_t)f * N;
    double a[5] = { 0.0, 0.0, 0.0, 0.0, 0.0 };
    for (size_t c = (size_t)blockIdx.x * 256 + threadIdx.x; c < N; c += (size_t)gridDim.x * 256) {
        int i, j, k;
        cell_ijk((unsigned)c, nx, ny, i, j, k);
        const double x = uf[c];
        a[0] += x;
        a[1] += x * x;
        a[2] += fabs(x);
        a[3] += fabs((double)tf[c]);
        const size_t row = (size_t)nx * (j + (size_t)ny * k);
        const double xp = uf[row + wrap1(i + 1, nx)], xm = uf[row + wrap1(i - 1, nx)];
        const double yp = uf[(size_t)i + (size_t)nx * (wrap1(j + 1, ny) + (size_t)ny * k)];
        const double ym = uf[(size_t)i + (size_t)nx * (wrap1(j - 1, ny) + (size_t)ny * k)];
        const double zp = uf[(size_t)i + (size_t)nx * (j + (size_t)ny * wrap1(k + 1, nz))];
        const double zm = uf[(size_t)i + (size_t)nx * (j + (size_t)ny * wrap1(k - 1, nz))];
        a[4] += fabs(xp - 2.0 * x + xm) + fabs(yp - 2.0 * x + ym) + fabs(zp - 2.0 * x + zm);
    }
    __shared__ double sh[5][256];
    for (int q = 0; q < 5; ++q) sh[q][threadIdx.x] = a[q];
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (threadIdx.x < st)
            for (int q = 0; q < 5; ++q) sh[q][threadIdx.x] += sh[q][threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x < 5) partial[((size_t)blockIdx.x * 8 + f) * 5 + threadIdx.x] = sh[threadIdx.x][0];
}

// out[q * 8 + f] = sum over blocks of partial[(b * 8 + f) * 5 + q]: 256
// threads over the blocks, then a fixed tree per output
__global__ void __launch_bounds__(256) stats_final_kernel(const double* __restrict__ partial, int nblk,
                                                          double* __restrict__ out)
{
    __shared__ double sh[256];
    for (int k = 0; k < 40; ++k) {
        const int q = k / 8, f = k % 8;
        double acc = 0.0;
        for (int b = threadIdx.x; b < nblk; b += 256) acc += partial[((size_t)b * 8 + f) * 5 + q];
        sh[threadIdx.x] = acc;
        __syncthreads();
        for (int st = 128; st > 0; st >>= 1) {
            if (threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
            __syncthreads();
        }
        if (threadIdx.x == 0) out[k] = sh[0];
        __syncthreads();
    }
}

hipError_t launch_stats(const float* u, const float* t, const int n[3], double* partial, double* out, hipStream_t s)
{
    hipLaunchKernelGGL(stats_partial_kernel, dim3(STATS_BLOCKS, 8), dim3(256), 0, s, u, t, n[0], n[1], n[2], partial);
    hipLaunchKernelGGL(stats_final_kernel, dim3(1), dim3(256), 0, s, partial, STATS_BLOCKS, out);
    return hipGetLastError();
}

// Roughness gate: g0(c) = (1/8) sum_f inv_R[f] * sum over axes
// |u_f(c+a) - 2 u_f(c) + u_f(c-a)| (u field-major FP32), and the network
// input x of normalize_kernel from the same loads.  A thread takes 4
// consecutive x cells (nx is a multiple of 4): one 16-byte load per field
// for the cells and for each y / z neighbour row, two scalars for x.
__global__ void __launch_bounds__(256) gate_rough_kernel(ClosureState u, int nx, int ny, int nz, GateScales gs,
                                                         ClosureScales sc, float* __restrict__ g0,
                                                         uint16_t* __restrict__ x)
{
    const unsigned N = (unsigned)nx * ny * nz, N4 = N / 4;
    for (unsigned t = blockIdx.x * blockDim.x + threadIdx.x; t < N4; t += gridDim.x * blockDim.x) {
        const unsigned c = 4 * t;
        int i, j, k;
        cell_ijk(c, nx, ny, i, j, k);
        const unsigned row = c - i;
        const unsigned cyp = (unsigned)i + (unsigned)nx * ((unsigned)wrap1(j + 1, ny) + (unsigned)ny * k);
        const unsigned cym = (unsigned)i + (unsigned)nx * ((unsigned)wrap1(j - 1, ny) + (unsigned)ny * k);
        const unsigned czp = (unsigned)i + (unsigned)nx * ((unsigned)j + (unsigned)ny * wrap1(k + 1, nz));
        const unsigned czm = (unsigned)i + (unsigned)nx * ((unsigned)j + (unsigned)ny * wrap1(k - 1, nz));
        const unsigned xm = row + wrap1(i - 1, nx), xp = row + wrap1(i + 4, nx);
        float acc[4] = { 0.f, 0.f, 0.f, 0.f };
        float b[4][8];
#pragma unroll
        for (int f = 0; f < 8; ++f) {
            const float* uf = field(u, f, N);
            const float4 v = *reinterpret_cast<const float4*>(uf + c);
            const float4 vyp = *reinterpret_cast<const float4*>(uf + cyp);
            const float4 vym = *reinterpret_cast<const float4*>(uf + cym);
            const float4 vzp = *reinterpret_cast<const float4*>(uf + czp);
            const float4 vzm = *reinterpret_cast<const float4*>(uf + czm);
            const float a[6] = { uf[xm], v.x, v.y, v.z, v.w, uf[xp] };
            const float yp[4] = { vyp.x, vyp.y, vyp.z, vyp.w }, ym[4] = { vym.x, vym.y, vym.z, vym.w };
            const float zp[4] = { vzp.x, vzp.y, vzp.z, vzp.w }, zm[4] = { vzm.x, vzm.y, vzm.z, vzm.w };
            const float w = gs.inv_r[f];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float x2 = 2.0f * a[q + 1];
                const float r = fabsf((a[q + 2] - x2) + a[q]) + fabsf((yp[q] - x2) + ym[q]) + fabsf((zp[q] - x2) + zm[q]);
                acc[q] += r * w;
                b[q][f] = (a[q + 1] - sc.in_mean[f]) / sc.in_std[f];
            }
        }
        *reinterpret_cast<float4*>(g0 + c) = make_float4(0.125f * acc[0], 0.125f * acc[1], 0.125f * acc[2], 0.125f * acc[3]);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<uint4*>(x + (size_t)(c + q) * 8) =
                make_uint4(f2bf2(b[q][0], b[q][1]), f2bf2(b[q][2], b[q][3]), f2bf2(b[q][4], b[q][5]), f2bf2(b[q][6], b[q][7]));
    }
}

// g(c) = max of g0 over c and its six face neighbours, 4 cells per thread
__global__ void __launch_bounds__(256) gate_max_kernel(const float* __restrict__ g0, int nx, int ny, int nz,
                                                       float* __restrict__ g)
{
    const unsigned N4 = (unsigned)nx * ny * nz / 4;
    for (unsigned t = blockIdx.x * blockDim.x + threadIdx.x; t < N4; t += gridDim.x * blockDim.x) {
        const unsigned c = 4 * t;
        int i, j, k;
        cell_ijk(c, nx, ny, i, j, k);
        const unsigned row = c - i;
        const unsigned near[4] = { (unsigned)i + (unsigned)nx * ((unsigned)wrap1(j + 1, ny) + (unsigned)ny * k),
                                   (unsigned)i + (unsigned)nx * ((unsigned)wrap1(j - 1, ny) + (unsigned)ny * k),
                                   (unsigned)i + (unsigned)nx * ((unsigned)j + (unsigned)ny * wrap1(k + 1, nz)),
                                   (unsigned)i + (unsigned)nx * ((unsigned)j + (unsigned)ny * wrap1(k - 1, nz)) };
        const float4 v = *reinterpret_cast<const float4*>(g0 + c);
        const float a[6] = { g0[row + wrap1(i - 1, nx)], v.x, v.y, v.z, v.w, g0[row + wrap1(i + 4, nx)] };
        float m[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) m[q] = fmaxf(fmaxf(a[q + 1], a[q + 2]), a[q]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float4 w = *reinterpret_cast<const float4*>(g0 + near[e]);
            m[0] = fmaxf(m[0], w.x); m[1] = fmaxf(m[1], w.y); m[2] = fmaxf(m[2], w.z); m[3] = fmaxf(m[3], w.w);
        }
        *reinterpret_cast<float4*>(g + c) = make_float4(m[0], m[1], m[2], m[3]);
    }
}

hipError_t launch_gate(const ClosureState& u, const int n[3], const GateScales& gs, const ClosureScales& sc, float* g0,
                       float* g, uint16_t* x, hipStream_t s)
{
    hipLaunchKernelGGL(gate_rough_kernel, dim3(2048), dim3(256), 0, s, u, n[0], n[1], n[2], gs, sc, g0, x);
    hipLaunchKernelGGL(gate_max_kernel, dim3(2048), dim3(256), 0, s, g0, n[0], n[1], n[2], g);
    return hipGetLastError();
}

}  // namespace mhd
