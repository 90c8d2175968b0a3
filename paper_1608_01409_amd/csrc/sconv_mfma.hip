// Layers that pruning left rather dense, on the matrix cores.
//
// Above a density of about a quarter most multiply-adds of a 32-row tile are real, and the matrix cores do dense
// arithmetic 20 times as fast as the vector units.  They have no fp32 format of that speed, so both operands are split
// into three bf16 parts, x = h + m + l exactly (3 x 8 significant bits), and the six products whose weight is 2^-16 or
// more are summed in fp32: h*h into one accumulator, h*m + m*h + m*m + h*l + l*h into a second one that is added at the
// end.  What is left out (m*l, l*m, l*l) is below 2^-24 of a product, where a fused multiply-add has the product exactly.
// One v_mfma_f32_32x32x16_bf16 adds 16 products with a few roundings (two halves of 2^-24 on top of 1 are lost one by one;
// denormals are carried in full), so the large accumulator is rounded a few times per 16 columns instead of once per
// nonzero.  Measured against fp64 per row of n stored nonzeros, relative error of the sums and largest error of an output in
// sum|w*x|, here / fp32 chain of the flat-stream kernel: n = 1 2.61e-8, 9.3e-8 / 2.53e-8, 6.0e-8; n = 2 2.71e-8, 1.75e-7 /
// 3.55e-8, 1.13e-7; n = 3 2.60e-8, 1.3e-7 / 3.93e-8, 1.6e-7; n = 16 3.3e-8, 1.35e-7 / 6.0e-8, 2.1e-7; n = 350 1.1e-7 / 1.8e-7.
// Rows of fewer than SCONV_MFMA_SHORT_ROW nonzeros are therefore summed over their nonzeros (n = 3 as a margin); layers in
// which they are more than a few stay on the sparse kernels.
//
// Activations are staged times 2^16 and weights packed times 2^-16.  The three parts then hold every activation below 2^111
// exactly, denormals included (the lowest bit of a float is 2^-149, that of a bf16 denormal 2^-133); weights are checked when
// they are packed.  Larger activations, infinities and NaN leave sums that are not finite, also where the weight they meet is
// a pruned one (a zero here).  A workgroup that finds such sums takes them again: a second pass leaves those activations out,
// a third has the large ones alone at another scale, a fourth counts which outputs have a stored weight on an infinity or NaN.
// 13x13, 384 -> 384 in two groups, 3x3, batch 256, density 0.5: 250-264 us with ordinary and with tiny activations, 695-770 us
// with infinities, NaN or values above 2^111 in every workgroup (flat-stream kernel 530; sums over the CSR arrays instead of
// the further passes took 40 ms).  1x1, 192 -> 64, 28x28, batch 64, density 0.3, through LDS: 21 and 61-85 us (flat-stream kernel 31).
//
// Implicit GEMM: rows = filters of a group, columns = output positions counted through the batch, depth = taps x
// channels.  A workgroup takes 32*MT filters and 128*NT positions and walks the channels in blocks of 8*g8.  The input
// rows its positions touch are staged once per block, split on the way, as [channel octet][cell][part][8 channels]: 16
// bytes are the 8 consecutive depths a lane feeds to an MFMA, whatever the tap, which only moves the cell; 48 bytes from
// cell to cell spread a wave's reads over all LDS banks.  Where four neighbouring cells are 16 consecutive bytes of the input a lane
// loads four cells x 8 channels in 8 loads: the address unit takes 16 clocks a load instruction whatever its width (45 random
// layers, 8-140 us: 1.064x, none slower by more than 1 %; two of them in flight at once cost the shapes with one accumulator
// tile a third of their waves and were 5-7 % slower there).  Weights are packed in fragment order and go from L2 straight to
// registers, one step ahead.  Two workgroups share a CU: one stages while the other multiplies.
//
// Measured: 13x13, 384 -> 384 in two groups, 3x3, batch 256, density 0.5: flat-stream kernel 530 us, here 250-264 us as the
// clocks allow, 344 GFLOP of bf16 products at 1.30-1.38 PFLOP/s (a large library product reaches 1.24).  Counters: matrix cores
// busy 59 % of the cycles, LDS bank conflicts 40 % of the LDS cycles, L2 hit rate 75 %.  Of 281 us at an earlier state staging
// was 37, weights from L2 instead of L1 10, bank conflicts 7.
#include <algorithm>
#include <type_traits>

#include "sconv_device.h"

namespace sconv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
using const_u32 = const __attribute__((address_space(4))) unsigned;
using const_i32 = const __attribute__((address_space(4))) int;

__device__ float mfma_buffer_load(int4v rsrc, int voffset, int soffset, int aux) __asm("llvm.amdgcn.raw.buffer.load.f32");

__device__ int4v mfma_buffer_load4(int4v rsrc, int voffset, int soffset, int aux) __asm("llvm.amdgcn.raw.buffer.load.v4i32");

#define INLINE __attribute__((always_inline))

struct MfmaArgs {
    const float *in;
    float *out;
    const bf16x8 *wfrag;     // [group][32-row tile][step][part][lane]
    const int *uoff;         // LDS byte offset of every depth octet, two per step: full block, then last block
    const int *choff;        // phase form: byte offset of a virtual channel relative to its group, else null
    const int *rowptr;       // the direct kernel's CSR, for workgroups that met a value the split cannot carry
    const uint32_t *trip;
    const float *bias;
    int relu;
    int P, OHW, OW, OH, H, W, Kg, pad, stride;
    int cstep, lstep;        // input elements per cell; cells per output position
    int Rr, Wl, row_img;     // filter rows in cells, cells per staged row, staged rows of a whole image
    int g8, nblk, steps, steps_last, total_steps, c_virtual;
    int plane;               // cells of a channel octet's plane in LDS
    int n_ptiles, n_mtiles, n_tiles32, groups;
    int splits, blk_split;   // workgroups along the channel blocks, blocks each of them takes
    long long split_stride;  // floats from one part's sums to the next (out then is the workspace)
    int in_ch4;              // bytes from one channel to the next
    long long in_img, in_group;   // floats from one image / one group's channels to the next
    long long in_floats;     // floats of the whole input
    long long out_img, out_row;
    int goff_mul;            // floats per unit of the CSR's offsets
    int short_rows;          // there are rows of 1 to SCONV_MFMA_SHORT_ROW - 1 nonzeros
    int wide;                // four neighbouring cells of a row are 16 consecutive bytes of the input
    int quads;               // fours of cells per row, the last one back by what it would pass the row's end
    FastDiv d_units, d_splits, d_mt, d_ohw, d_ow, d_wl, d_rowimg, d_quads;
};

// Division of an item number (below 320) by the number of pieces, at most 16: ceil(2^32 / pieces), 0 for 1.  (A table among the
// arguments, indexed in the kernel, puts all of them into scratch memory once they are used in many places.)
#define SCONV_MAGIC(D) 0xffffffffu / D + 1u
static __constant__ unsigned kPieceMagic[17] = {0, 0, SCONV_MAGIC(2), SCONV_MAGIC(3), SCONV_MAGIC(4), SCONV_MAGIC(5), SCONV_MAGIC(6), SCONV_MAGIC(7),
    SCONV_MAGIC(8), SCONV_MAGIC(9), SCONV_MAGIC(10), SCONV_MAGIC(11), SCONV_MAGIC(12), SCONV_MAGIC(13), SCONV_MAGIC(14), SCONV_MAGIC(15), SCONV_MAGIC(16)};
#undef SCONV_MAGIC

static __device__ __forceinline__ void split8(const float (&x)[8], uint4 &h, uint4 &m, uint4 &l)
{
    unsigned hw[4], mw[4], lw[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const f32x2 v = {x[2 * i] * SCONV_MFMA_SCALE, x[2 * i + 1] * SCONV_MFMA_SCALE};
        const bf16x2 hb = __builtin_convertvector(v, bf16x2);
        hw[i] = __builtin_bit_cast(unsigned, hb);
        const f32x2 r = {v[0] - __uint_as_float(hw[i] << 16), v[1] - __uint_as_float(hw[i] & 0xffff0000u)};
        const bf16x2 mb = __builtin_convertvector(r, bf16x2);
        mw[i] = __builtin_bit_cast(unsigned, mb);
        const f32x2 q = {r[0] - __uint_as_float(mw[i] << 16), r[1] - __uint_as_float(mw[i] & 0xffff0000u)};
        const bf16x2 lb = __builtin_convertvector(q, bf16x2);
        lw[i] = __builtin_bit_cast(unsigned, lb);
    }
    h = make_uint4(hw[0], hw[1], hw[2], hw[3]);
    m = make_uint4(mw[0], mw[1], mw[2], mw[3]);
    l = make_uint4(lw[0], lw[1], lw[2], lw[3]);
}

static __device__ __forceinline__ bool not_finite(float v) { return (__float_as_uint(v) & 0x7f800000u) == 0x7f800000u; }
// too large for the split, infinities and NaN included: 2^111
static __device__ __forceinline__ bool too_large(float v) { return (__float_as_uint(v) & 0x7fffffffu) >= 0x77000000u; }

// The infinities and NaN among eight activations: 1 in h where a positive one is (a NaN is both), 1 in m where a negative one
static __device__ __forceinline__ void marks8(const float (&x)[8], uint4 &h, uint4 &m)
{
    unsigned hw[4], mw[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        hw[i] = mw[i] = 0;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const float v = x[2 * i + e];
            if (v == __builtin_inff() || v != v) hw[i] |= 0x3f80u << (16 * e);
            if (v == -__builtin_inff() || v != v) mw[i] |= 0x3f80u << (16 * e);
        }
    }
    h = make_uint4(hw[0], hw[1], hw[2], hw[3]);
    m = make_uint4(mw[0], mw[1], mw[2], mw[3]);
}

// Output (k, position p) over the stored nonzeros of a short row, as the direct kernel sums them.
static __device__ __forceinline__ float row_sum(const MfmaArgs &a, int k, int p)
{
    const int n = p / a.OHW, q = p - n * a.OHW, y = q / a.OW * a.stride, x = q % a.OW * a.stride;
    const float *im = a.in + n * a.in_img;
    float v = 0.f;
    for (int j = a.rowptr[k]; j < a.rowptr[k + 1]; ++j) {
        const int goff = (int)a.trip[3 * (size_t)j + 1];
        const uint32_t rs = a.trip[3 * (size_t)j + 2];
        const int iy = y + (int)(short)(rs >> 16), ix = x + (int)(short)(rs & 0xffffu);
        const bool inside = iy >= 0 && iy < a.H && ix >= 0 && ix < a.W;
        const float xv = inside ? im[(y * a.W + x + goff) * (long long)a.goff_mul] : 0.f;
        v = fmaf(__uint_as_float(a.trip[3 * (size_t)j]), xv, v);
    }
    return v;
}

// What a workgroup works on.  Workgroup ids go round the 8 XCDs.  Position tiles are taken 8 at a time, one per XCD, so that
// the workgroups that stage the same positions for different filters meet in one L2; the tiles left over are spread over all
// XCDs unit by unit (169 tiles x 6 units on one XCD more than on the others cost that XCD a third round).
struct Tile {
    int ptile, split, g, mt;
};
static __device__ __forceinline__ Tile tile_of(const MfmaArgs &a, int bid)
{
    const int units = a.n_mtiles * a.groups * a.splits, full = (a.n_ptiles >> 3) * 8 * units;
    Tile t;
    int unit;
    if (bid < full) {
        const int slot = bid >> 3, sq = fdiv(slot, a.d_units);
        unit = slot - sq * units;
        t.ptile = sq * 8 + (bid & 7);
    } else {
        const int sq = fdiv(bid - full, a.d_units);
        unit = bid - full - sq * units;
        t.ptile = (a.n_ptiles >> 3) * 8 + sq;
    }
    const int um = fdiv(unit, a.d_splits);
    t.split = unit - um * a.splits;
    t.g = fdiv(um, a.d_mt);
    t.mt = um - t.g * a.n_mtiles;
    return t;
}

// Four neighbouring cells x 8 channels on their way into LDS, and where they go (all ones: nowhere).
struct Four {
    f32x4 x[8];
    unsigned at;
};

// again = false: a workgroup's sums, stored with the epilogue, or without it and true if some are not finite.
// again = true: those sums once more (see above).
template <int MT, int NT, bool again>
static __device__ __forceinline__ bool multiply_tile(const MfmaArgs &a, const Tile &tile, char *lds)
{
    constexpr int kBatch = 4;
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int ptile = tile.ptile, split = tile.split, g = tile.g, mt = tile.mt;
    const int b_first = split * a.blk_split, b_end = min(b_first + a.blk_split, a.nblk);   // this workgroup's channel blocks

    const int p0 = ptile * (128 * NT);
    const int n_first = fdiv(p0, a.d_ohw), y_first = fdiv(p0 - n_first * a.OHW, a.d_ow);
    const int rows_first = (a.OH - 1 - y_first) * a.lstep + a.Rr;      // staged rows of the first image
    auto row_of = [&](int n, int y) {
        return n == n_first ? (y - y_first) * a.lstep : rows_first + (n - n_first - 1) * a.row_img + y * a.lstep;
    };
    int cells;
    {
        const int p1 = min(p0 + 128 * NT, a.P) - 1;
        const int n = fdiv(p1, a.d_ohw), y = fdiv(p1 - n * a.OHW, a.d_ow);
        cells = (row_of(n, y) + a.Rr) * a.Wl;
    }
    // where this lane's positions sit
    unsigned lane_addr[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int p = min(p0 + (wave * NT + t) * 32 + (lane & 31), a.P - 1);
        const int n = fdiv(p, a.d_ohw), q = p - n * a.OHW, y = fdiv(q, a.d_ow), x = q - y * a.OW;
        lane_addr[t] = (unsigned)(row_of(n, y) * a.Wl + x * a.lstep) * 48u;
    }
    // where the cells come from, relative to image n_first (a table in LDS behind the staged block and the depth octets'
    // offsets): padding and cells past the end read beyond the buffer
    const int n_off = 2 * (a.steps + a.steps_last);
    int *tbl = reinterpret_cast<int *>(lds + (size_t)a.g8 * a.plane * 48);
    unsigned *voff = reinterpret_cast<unsigned *>(tbl + n_off);
    // wide: per four of cells also where they go in LDS; what no four covers is padding and stays zero
    uint2 *four = reinterpret_cast<uint2 *>(voff);
    const bool wide = !again && a.wide;
    const int n_fours = wide ? fdiv(cells, a.d_wl) * a.quads : 0;
    if (wide)
        for (int i = threadIdx.x; i < a.g8 * a.plane * 3; i += 256) reinterpret_cast<uint4 *>(lds)[i] = make_uint4(0, 0, 0, 0);
    for (int i = threadIdx.x; i < (wide ? n_fours : a.plane); i += 256) {
        int row, col;            // of the cell, or of the first of four
        if (wide) {
            row = fdiv(i, a.d_quads);
            col = a.pad + min((i - row * a.quads) * 4, a.W - 4);
        } else {
            row = fdiv(i, a.d_wl);
            col = i - row * a.Wl;
        }
        int n = 0, yp = y_first * a.lstep + row;
        if (row >= rows_first) {
            const int img = fdiv(row - rows_first, a.d_rowimg);
            n = 1 + img;
            yp = row - rows_first - img * a.row_img;
        }
        const int iy = yp * a.cstep - a.pad, ix = col * a.cstep - a.pad;
        const bool ok = (wide || i < cells) && iy >= 0 && iy < a.H && ix >= 0 && ix < a.W;
        const unsigned from = ok ? (unsigned)(n * (int)a.in_img + iy * a.W + ix) * 4u : 0x80000000u;
        if (wide) four[i] = make_uint2(from, ok ? (unsigned)(row * a.Wl + col) * 48u : 0xffffffffu);
        else voff[i] = from;
    }
    const FastDiv d_fours = {(unsigned)n_fours, n_fours > 1 ? 0xffffffffu / (unsigned)n_fours + 1u : 0u};
    for (int i = threadIdx.x; i < n_off; i += 256) tbl[i] = a.uoff[i];
    const int pieces = (cells + 63) >> 6;
    const FastDiv d_pieces = {(unsigned)pieces, ((const_u32 *)kPieceMagic)[pieces]};
    const float *src = a.in + n_first * a.in_img + g * a.in_group;
    int4v rsrc;
    {
        const unsigned long long ip = (unsigned long long)src;
        const long long left = (a.in_floats - (n_first * a.in_img + g * a.in_group)) * 4;
        rsrc.x = __builtin_amdgcn_readfirstlane((int)(unsigned)ip);
        rsrc.y = __builtin_amdgcn_readfirstlane((int)(unsigned)(ip >> 32));
        rsrc.z = __builtin_amdgcn_readfirstlane((int)min(left, 0x7fffffffll));
        rsrc.w = 0x00020000;
    }

    f32x16 acc[MT][NT], cor[MT][NT];

    // weights: step by step from a scalar offset per row tile; the fragments end with a spare step
    int4v wrsrc;
    {
        const unsigned long long wp = (unsigned long long)(a.wfrag + (size_t)(g * a.n_tiles32 + mt * MT) * a.total_steps * 192);
        wrsrc.x = __builtin_amdgcn_readfirstlane((int)(unsigned)wp);
        wrsrc.y = __builtin_amdgcn_readfirstlane((int)(unsigned)(wp >> 32));
        wrsrc.z = __builtin_amdgcn_readfirstlane((MT * a.total_steps + 1) * 3072);
        wrsrc.w = 0x00020000;
    }
    const int lane16 = lane * 16;
    int wstep = 0;
    auto load_a = [&](bf16x8 (&A)[MT][3]) INLINE {
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int s = 0; s < 3; ++s)
                A[m][s] = __builtin_bit_cast(bf16x8, mfma_buffer_load4(wrsrc, lane16 + s * 1024, m * a.total_steps * 3072 + wstep, 0));
        wstep += 3072;
    };
    auto load_b = [&](bf16x8 (&B)[NT][3], unsigned off) INLINE {
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
            for (int t = 0; t < NT; ++t) B[t][s] = *reinterpret_cast<const bf16x8 *>(lds + lane_addr[t] + off + s * 16);
    };
    auto multiply = [&](const bf16x8 (&A)[MT][3], const bf16x8 (&B)[NT][3]) INLINE {
#define SCONV_MFMA(D, PA, PB) \
    _Pragma("unroll") for (int m = 0; m < MT; ++m) \
        _Pragma("unroll") for (int t = 0; t < NT; ++t) \
            D[m][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[m][PA], B[t][PB], D[m][t], 0, 0, 0);
        SCONV_MFMA(acc, 0, 0)
        SCONV_MFMA(cor, 1, 0)
        SCONV_MFMA(cor, 2, 0)
        SCONV_MFMA(cor, 0, 1)
        SCONV_MFMA(cor, 1, 1)
        SCONV_MFMA(cor, 0, 2)
#undef SCONV_MFMA
    };
    // stored weights on infinities: acc counts products that are +infinity, cor those that are -infinity (a stored zero, -0
    // here, makes NaN of either and counts as both)
    auto count = [&](const bf16x8 (&A)[MT][3], const bf16x8 (&B)[NT][3]) INLINE {
        bf16x8 S[MT][2];
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const s16x8 w = __builtin_bit_cast(s16x8, A[m][0]);
            S[m][0] = __builtin_bit_cast(bf16x8, (s16x8)(((w > 0) | (w == (short)0x8000)) & (short)0x3f80));
            S[m][1] = __builtin_bit_cast(bf16x8, (s16x8)((w < 0) & (short)0x3f80));
        }
#define SCONV_MFMA(D, PA, PB) \
    _Pragma("unroll") for (int m = 0; m < MT; ++m) \
        _Pragma("unroll") for (int t = 0; t < NT; ++t) \
            D[m][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(S[m][PA], B[t][PB], D[m][t], 0, 0, 0);
        SCONV_MFMA(acc, 0, 0)
        SCONV_MFMA(acc, 1, 1)
        SCONV_MFMA(cor, 1, 0)
        SCONV_MFMA(cor, 0, 1)
#undef SCONV_MFMA
    };
    bf16x8 A[MT][3];
    bool seen_large = false, seen_inf = false;     // by kSplit: finite values it left out, infinities or NaN
    const_i32 *choff = (const_i32 *)a.choff;

    // One pass over this workgroup's channel blocks: kAll activations, kSplit those that the split holds, kLarge the other
    // finite ones times 2^-32, kCount (see count).
    enum Mode { kAll, kSplit, kLarge, kCount };
    auto pass = [&](auto mode_) INLINE {
        constexpr Mode mode = decltype(mode_)::value;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[m][t][r] = cor[m][t][r] = 0.f;
        wstep = b_first * a.steps * 3072;
        load_a(A);
        auto use = [&](const bf16x8 (&A)[MT][3], const bf16x8 (&B)[NT][3]) INLINE {
            if constexpr (mode == kCount)
                count(A, B);
            else
                multiply(A, B);
        };
        auto load_four = [&](Four &v, int b, int i0, int fours) INLINE {
            const int i = min(i0 + lane, fours - 1), o = fdiv(i, d_fours);
            const uint2 e = four[i - o * n_fours];
            const int c = (b * a.g8 + o) * 8;
            v.at = i0 + lane < fours && e.y != 0xffffffffu ? e.y + (unsigned)(o * a.plane) * 48u : 0xffffffffu;
            const unsigned vo = i0 + lane < fours ? e.x + (unsigned)(c * a.in_ch4) : 0x80000000u;
#pragma unroll
            for (int q = 0; q < 8; ++q)
                v.x[q] = __builtin_bit_cast(f32x4, mfma_buffer_load4(rsrc, (int)(c + q < a.c_virtual ? vo + (unsigned)(q * a.in_ch4) : 0x80000000u), 0, 0));
            __builtin_amdgcn_sched_barrier(0);
        };
        auto store_four = [&](const Four &v) INLINE {
            if (v.at != 0xffffffffu) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x[8] = {v.x[0][e], v.x[1][e], v.x[2][e], v.x[3][e], v.x[4][e], v.x[5][e], v.x[6][e], v.x[7][e]};
                    uint4 h, m, l;
                    split8(x, h, m, l);
                    uint4 *dst = reinterpret_cast<uint4 *>(lds + v.at + e * 48);
                    dst[0] = h;
                    dst[1] = m;
                    dst[2] = l;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        if (wide) __syncthreads();           // the table is there
        for (int b = b_first; b < b_end; ++b) {
            if (mode == kAll && wide) {
                // items of 64 lanes, four cells x 8 channels each, counted through the block's octets
                const int fours = min(a.g8, (a.c_virtual - b * a.g8 * 8 + 7) >> 3) * n_fours;
                Four v;
                load_four(v, b, wave * 64, fours);
                __syncthreads();             // the block before is used up
                for (int i0 = wave * 64; i0 < fours; i0 += 256) {
                    if (i0 >= 256) load_four(v, b, i0, fours);
                    store_four(v);
                }
            } else {
                __syncthreads();
                // items of 64 cells x 8 channels, dealt to the waves; the loads of four items are in flight together
                const int c0 = b * a.g8 * 8, items = min(a.g8, (a.c_virtual - c0 + 7) >> 3) * pieces;
                for (int i0 = wave; i0 < items; i0 += 4 * kBatch) {
                    float x[kBatch][8];
#pragma unroll
                    for (int j = 0; j < kBatch; ++j) {
                        const int item = min(i0 + 4 * j, items - 1), o = fdiv(item, d_pieces), piece = item - o * pieces, c = c0 + o * 8;
                        const unsigned vo = i0 + 4 * j < items ? voff[piece * 64 + lane] : 0x80000000u;
                        int co[8];
                        if (a.choff) {
#pragma unroll
                            for (int i = 0; i < 8; ++i) co[i] = choff[c + i];
                        } else {
#pragma unroll
                            for (int i = 0; i < 8; ++i) co[i] = c + i < a.c_virtual ? (c + i) * a.in_ch4 : SCONV_MFMA_NO_CHANNEL;
                        }
#pragma unroll
                        for (int i = 0; i < 8; ++i)        // a channel past the last one reads beyond the buffer's end: 0
                            x[j][i] = mfma_buffer_load(rsrc, (int)(vo | ((unsigned)co[i] & 0x80000000u)), co[i] & 0x7fffffff, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int j = 0; j < kBatch; ++j) {
                        const int item = i0 + 4 * j, o = fdiv(item, d_pieces), piece = item - o * pieces;
                        if (item >= items) break;
                        uint4 h, m, l;
                        if constexpr (mode == kCount) {
                            marks8(x[j], h, m);
                            l = make_uint4(0, 0, 0, 0);
                        } else {
#pragma unroll
                            for (int i = 0; mode != kAll && i < 8; ++i) {
                                const float v = x[j][i];
                                const bool inf = not_finite(v), large = too_large(v) && !inf;
                                seen_inf |= inf;
                                seen_large |= large;
                                x[j][i] = mode == kLarge ? (large ? v * 0x1p-32f : 0.f) : (inf || large ? 0.f : v);
                            }
                            split8(x[j], h, m, l);
                        }
                        uint4 *dst = reinterpret_cast<uint4 *>(lds + ((size_t)o * a.plane + piece * 64 + lane) * 48);
                        dst[0] = h;
                        dst[1] = m;
                        dst[2] = l;
                    }
                }
            }
            __syncthreads();
            // the weights of the next step are on their way while one is multiplied
            const bool last = b == a.nblk - 1;
            const int *u = tbl + half + (last ? 2 * a.steps : 0); // lanes 0-31 take the even octets, lanes 32-63 the odd ones
            const int steps = last ? a.steps_last : a.steps;
            bf16x8 B0[NT][3], B1[NT][3], A1[MT][3];
            load_b(B0, (unsigned)u[0]);
            unsigned off = (unsigned)u[2 * min(1, steps - 1)];
            int i = 0;
            for (; i + 1 < steps; i += 2) {
                load_a(A1);
                load_b(B1, off);
                off = (unsigned)u[2 * min(i + 2, steps - 1)];
                __builtin_amdgcn_sched_barrier(0);
                use(A, B0);
                __builtin_amdgcn_sched_barrier(0);
                load_a(A);
                load_b(B0, off);
                off = (unsigned)u[2 * min(i + 3, steps - 1)];
                __builtin_amdgcn_sched_barrier(0);
                use(A1, B1);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (i < steps) {
                load_a(A1);
                __builtin_amdgcn_sched_barrier(0);
                use(A, B0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int s = 0; s < 3; ++s) A[m][s] = A1[m][s];
            }
        }
    };

    // any(x): whether x holds in one of the workgroup's threads (through LDS, over the staged block)
    volatile int *flag = reinterpret_cast<volatile int *>(lds);
    auto any = [&](bool x) INLINE {
        __syncthreads();
        if (threadIdx.x == 0) *flag = 0;
        __syncthreads();
        if (x) *flag = 1;
        __syncthreads();
        return *flag != 0;
    };
    // f(output, row, sum) for every output of this lane
    auto outputs = [&](auto f) INLINE {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int p = p0 + (wave * NT + t) * 32 + (lane & 31);
            if (p >= a.P) continue;
            const int n = fdiv(p, a.d_ohw);
            float *dst = a.out + split * a.split_stride + n * a.out_img + (p - n * a.OHW);
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int kl = (mt * MT + m) * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                    if (kl >= a.Kg) continue;
                    const int k = g * a.Kg + kl;
                    f(dst[k * a.out_row], k, acc[m][t][r], cor[m][t][r]);
                }
        }
    };
    auto finish = [&](float v, int k) INLINE {
        if (a.bias) v += a.bias[k];
        return a.relu ? fmaxf(v, 0.f) : v;
    };
    bool bad = false;
    if constexpr (!again) {
        pass(std::integral_constant<Mode, kAll>{});
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    acc[m][t][r] += cor[m][t][r];
                    bad |= not_finite(acc[m][t][r]);
                }
        bad = any(bad);
        const bool bias = a.bias && !bad, relu = a.relu && !bad;
        outputs([&](float &out, int k, float v, float) INLINE {
            if (bias) v += a.bias[k];
            out = relu ? fmaxf(v, 0.f) : v;
        });
    } else {
        // (through the output: there is no room for a second set of accumulators)
        pass(std::integral_constant<Mode, kSplit>{});
        outputs([&](float &out, int, float v, float c) INLINE {
            if (not_finite(out)) out = v + c;
        });
        if (any(seen_large)) {
            pass(std::integral_constant<Mode, kLarge>{});
            outputs([&](float &out, int, float v, float c) INLINE { out += (v + c) * 0x1p32f; });
        }
        if (any(seen_inf)) {
            pass(std::integral_constant<Mode, kCount>{});
            outputs([&](float &out, int, float up, float down) INLINE {
                if (up > 0.f) out += __builtin_inff();
                if (down > 0.f) out -= __builtin_inff();
            });
        }
        if (a.bias || a.relu)
            outputs([&](float &out, int k, float, float) INLINE {
                const float v = a.bias ? out + a.bias[k] : out;
                out = a.relu ? fmaxf(v, 0.f) : v;
            });
    }
    return bad;
}

// The short rows of a workgroup, over what it has stored; of several parts the first holds the whole sum.
template <int MT, int NT>
static __device__ __forceinline__ void sum_short_rows(const MfmaArgs &a, const Tile &t)
{
    const int lane = threadIdx.x & 63;
    const int kl = t.mt * MT * 32 + lane, row = t.g * a.Kg + min(kl, a.Kg - 1), nnz = a.rowptr[row + 1] - a.rowptr[row];
    unsigned long long rows = __ballot(lane < 32 * MT && kl < a.Kg && nnz > 0 && nnz < SCONV_MFMA_SHORT_ROW);
    __syncthreads();
    for (; rows; rows &= rows - 1) {
        const int k = t.g * a.Kg + t.mt * MT * 32 + __ffsll(rows) - 1, p = t.ptile * (128 * NT) + (int)threadIdx.x;
        if ((int)threadIdx.x >= 128 * NT || p >= a.P) continue;
        const int n = p / a.OHW;
        float v = t.split == 0 ? row_sum(a, k, p) : 0.f;
        if (a.bias) v += a.bias[k];
        if (a.relu) v = fmaxf(v, 0.f);
        a.out[t.split * a.split_stride + n * a.out_img + k * a.out_row + (p - n * a.OHW)] = v;
    }
}

// What is left to do for a few workgroups: sums that were not finite, short rows.
template <int MT, int NT>
static __device__ __forceinline__ void finish_tile(const MfmaArgs &a, bool bad, char *lds)
{
    if (!bad && !a.short_rows) return;
    // The rare rest reads the arguments again, out of the compiler's sight: with their values kept for it the first pass spills
    // scalar registers (13x13, 384 -> 384 in two groups, density 0.5, batch 256: 263 us instead of 251).
    unsigned long long args = (unsigned long long)__builtin_amdgcn_kernarg_segment_ptr();
    int bid = blockIdx.x;
    asm volatile("" : "+s"(args), "+s"(bid));
    const MfmaArgs &b = *(const MfmaArgs *)(const __attribute__((address_space(4))) MfmaArgs *)args;
    const Tile tile = tile_of(b, bid);
    if (bad) multiply_tile<MT, NT, true>(b, tile, lds);
    if (b.short_rows) sum_short_rows<MT, NT>(b, tile);
}

template <int MT, int NT>
__global__ void __launch_bounds__(256, 2) sconv_mfma_kernel(const MfmaArgs a)
{
    extern __shared__ uint4 smem[];
    char *lds = reinterpret_cast<char *>(smem);
    const bool bad = multiply_tile<MT, NT, false>(a, tile_of(a, blockIdx.x), lds);
    finish_tile<MT, NT>(a, bad, lds);
}

// Layers of one tap at stride 1, fully connected ones among them (sconv_mfma_column_kernel).  No activation is used at two
// positions of a workgroup, so LDS saves no load: a lane loads the 8 channels x 1 position that it feeds to the matrix instruction,
// with the same split, the same products and the same order of them as above (same bits).  No barrier, no table; a step's loads are
// asked for two steps before, in straight code: where a branch may leave some out the compiler waits for more of them than a step
// needs (16.2 us for 15.2), so a last step of fewer than 16 channels (kShort) has registers of its own, loaded at the beginning.
// What bounds it: the address unit is the busiest (14 load instructions a wave and step, 14 clocks each, where the matrix cores need
// 384 / 4), for 33 % of the first layer's launch on average, 42 % on a CU with two workgroups (matrix cores 13 %); the rest is one round of few
// waves: launch, first loads, stores.  192 -> 64, 28x28, batch 64, density 0.3: through LDS 20.5 us, here 15.2 (floor 10); 512 -> 128,
// 28x28, batch 32: 35.0 -> 25.5; 512 -> 512, 14x14, batch 64: 64.0 -> 48.9; fully connected 2048 -> 512, batch 256: 18.7 -> 13.8.
// Not taken: weights through LDS, two steps at a time (a barrier every two steps: 17.8 us in the first layer), loads four steps ahead (16.3),
// two positions a lane (18.0; 512 -> 512 44.8), 128 filters a wave (23.3).
template <int MT, bool kShort>
static __device__ __forceinline__ bool column_tile(const MfmaArgs &a, const Tile &tile, char *lds)
{
    constexpr int D = 2;                     // steps loaded ahead (even: the split activations alternate)
    const int lane = threadIdx.x & 63, half = lane >> 5, lane16 = lane * 16;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    volatile int *flag = reinterpret_cast<volatile int *>(lds);
    if (threadIdx.x == 0) *flag = 0;
    const int b_first = tile.split * a.blk_split, b_end = min(b_first + a.blk_split, a.nblk);
    const int first_step = b_first * a.steps, total = (b_end - b_first) * a.steps - (b_end == a.nblk ? a.steps - a.steps_last : 0);
    const int full = kShort ? min(total, a.c_virtual / 16 - first_step) : total;   // steps of 16 channels; one of fewer may follow
    const int p0 = tile.ptile * 128, n_first = fdiv(p0, a.d_ohw), p = p0 + wave * 32 + (lane & 31);
    const int n = fdiv(min(p, a.P - 1), a.d_ohw), q = min(p, a.P - 1) - n * a.OHW;
    const bool there = p < a.P;
    int4v rsrc, wrsrc;
    {
        const long long first = n_first * a.in_img + tile.g * a.in_group;
        const unsigned long long ip = (unsigned long long)(a.in + first);
        rsrc.x = __builtin_amdgcn_readfirstlane((int)(unsigned)ip);
        rsrc.y = __builtin_amdgcn_readfirstlane((int)(unsigned)(ip >> 32));
        rsrc.z = __builtin_amdgcn_readfirstlane((int)min((a.in_floats - first) * 4, 0x7fffffffll));
        rsrc.w = 0x00020000;
    }
    {
        const size_t first = (size_t)(tile.g * a.n_tiles32 + tile.mt * MT) * a.total_steps + first_step;
        const unsigned long long wp = (unsigned long long)(a.wfrag + first * 192);
        wrsrc.x = __builtin_amdgcn_readfirstlane((int)(unsigned)wp);
        wrsrc.y = __builtin_amdgcn_readfirstlane((int)(unsigned)(wp >> 32));
        wrsrc.z = __builtin_amdgcn_readfirstlane(((MT - 1) * a.total_steps + total) * 3072);
        wrsrc.w = 0x00020000;
    }
    // (a position past the last one reads beyond the buffer's end: 0)
    const unsigned from = (there ? (unsigned)((n - n_first) * (int)a.in_img + q) * 4u : 0x80000000u) + (unsigned)(half * 8 * a.in_ch4);
    struct X {
        float v[8];
    };
    bf16x8 A[D][MT][3], B[2][3];
    X x[D], tail;
    int x_step = 0, a_step = 0;              // asked for next; past the last one that one again
    // (without a full step its first channel eight times, not used: the others may not exist)
    const int last = kShort ? max(full - 1, 0) : full - 1, ch4 = kShort && full == 0 ? 0 : a.in_ch4;
    auto load_x = [&](X &x) INLINE {
        int so = (first_step + min(x_step, last)) * 16 * a.in_ch4;
#pragma unroll
        for (int i = 0; i < 8; ++i, so += ch4) x.v[i] = mfma_buffer_load(rsrc, (int)from, so, 0);
        ++x_step;
    };
    auto load_a = [&](bf16x8 (&A)[MT][3]) INLINE {
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int s = 0; s < 3; ++s)
                A[m][s] = __builtin_bit_cast(bf16x8, mfma_buffer_load4(wrsrc, lane16 + s * 1024, (m * a.total_steps + min(a_step, total - 1)) * 3072, 0));
        ++a_step;
    };
    auto split = [&](bf16x8 (&B)[3], const X &x) INLINE {
        uint4 h, m, l;
        split8(x.v, h, m, l);
        B[0] = __builtin_bit_cast(bf16x8, h);
        B[1] = __builtin_bit_cast(bf16x8, m);
        B[2] = __builtin_bit_cast(bf16x8, l);
    };
    f32x16 acc[MT], cor[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[m][r] = cor[m][r] = 0.f;
    auto multiply = [&](const bf16x8 (&A)[MT][3], const bf16x8 (&B)[3]) INLINE {
#define SCONV_MFMA(D, PA, PB) \
    _Pragma("unroll") for (int m = 0; m < MT; ++m) D[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[m][PA], B[PB], D[m], 0, 0, 0);
        SCONV_MFMA(acc, 0, 0)
        SCONV_MFMA(cor, 1, 0)
        SCONV_MFMA(cor, 2, 0)
        SCONV_MFMA(cor, 0, 1)
        SCONV_MFMA(cor, 1, 1)
        SCONV_MFMA(cor, 0, 2)
#undef SCONV_MFMA
    };
#pragma unroll
    for (int j = 0; j < D; ++j) {
        load_x(x[j]);
        load_a(A[j]);
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (kShort) {
        const int c0 = (first_step + full) * 16, limit = full < total ? a.c_virtual : 0;
#pragma unroll
        for (int i = 0; i < 8; ++i)          // a channel past the last one: 0
            tail.v[i] = mfma_buffer_load(rsrc, (int)(c0 + i + 8 * half < limit ? from : 0x80000000u), c0 + i < limit ? (c0 + i) * a.in_ch4 : 0, 0);
    }
    split(B[0], x[0]);
    load_x(x[0]);
    __builtin_amdgcn_sched_barrier(0);
    // (the next step's activations are split between this step's matrix instructions)
    auto step = [&](int j) INLINE {
        split(B[(j + 1) & 1], x[(j + 1) % D]);
        multiply(A[j], B[j & 1]);
        __builtin_amdgcn_sched_barrier(0);
        load_x(x[(j + 1) % D]);
        load_a(A[j]);
        __builtin_amdgcn_sched_barrier(0);
    };
    int i = 0;
    for (; i + D <= full; i += D) {
#pragma unroll
        for (int j = 0; j < D; ++j) step(j);
    }
    const int left = full - i;
#pragma unroll
    for (int j = 0; j < D - 1; ++j)
        if (left > j) step(j);
    if (kShort && full < total) {
        bf16x8 T[3];
        split(T, tail);
#pragma unroll
        for (int j = 0; j < D; ++j)
            if (left == j) multiply(A[j], T);
    }
    const int k0 = tile.g * a.Kg + tile.mt * (MT * 32), rows = a.Kg - tile.mt * (MT * 32) - 4 * half;  // rows: this lane's, counted as below
    const bool whole = a.Kg >= (tile.mt + 1) * (MT * 32);
    // The bias is there before the first sum is stored: loaded between the stores, row by row, each of them waited for the stores before
    // it (57 -> 400, 55x55, batch 17: 70.3 us; now 50.4).
    float4u add[MT][4];
    if (a.bias) {
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float *from = a.bias + k0 + 4 * half;
                if (whole) add[m][i] = *reinterpret_cast<const float4u *>(from + m * 32 + 8 * i);
                else
#pragma unroll
                    for (int e = 0; e < 4; ++e) add[m][i][e] = from[min(m * 32 + 8 * i + e, rows - 1)];   // (rows - 1 is the group's last)
            }
    }
    float zero = 0.f;                        // NaN once a sum is not finite
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            acc[m][r] += cor[m][r];
            zero = __builtin_fmaf(acc[m][r], 0.f, zero);
        }
    __syncthreads();                         // (the flag is cleared)
    if (zero != 0.f) *flag = 1;
    __syncthreads();
    const bool bad = *flag != 0, bias = a.bias && !bad, relu = a.relu && !bad;
    char *base = reinterpret_cast<char *>(a.out + tile.split * a.split_stride + n_first * a.out_img + k0 * a.out_row);
    const unsigned at = (unsigned)((n - n_first) * (int)a.out_img + q + 4 * half * (int)a.out_row) * 4u;
    if (there) {
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int kl = m * 32 + 8 * (r >> 2) + (r & 3);
                if (!whole && kl >= rows) continue;
                float v = acc[m][r];
                if (bias) v += add[m][r >> 2][r & 3];
                *reinterpret_cast<float *>(base + kl * a.out_row * 4 + at) = relu ? fmaxf(v, 0.f) : v;
            }
    }
    return bad;
}

template <int MT, bool kShort>
__global__ void __launch_bounds__(256, 2) sconv_mfma_column_kernel(const MfmaArgs a)
{
    extern __shared__ uint4 smem[];
    char *lds = reinterpret_cast<char *>(smem);
    const bool bad = column_tile<MT, kShort>(a, tile_of(a, blockIdx.x), lds);
    finish_tile<MT, 1>(a, bad, lds);
}

static int launch_mfma_inst(void (*kern)(const MfmaArgs), const MfmaArgs &a, int grid, int lds_bytes, hipStream_t s, int *hip_err)
{
    const int rc = allow_full_lds(reinterpret_cast<const void *>(kern), hip_err);
    if (rc) return rc;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(256), lds_bytes, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        *hip_err = (int)e;
        return SCONV_ERR_HIP;
    }
    return SCONV_OK;
}

int launch_mfma(const sconv_desc &layer, const MfmaTiling &t, const DeviceMfma &dev, const DeviceDirect &direct, const float *in, float *out,
                int N, bool feature_major, const Epilogue &ep, int64_t split_stride, void *stream, int *hip_err)
{
    const sconv_desc d = mfma_desc(layer);
    const Geometry g = geometry(d);
    MfmaArgs a;
    a.in = in;
    a.out = out;
    a.wfrag = static_cast<const bf16x8 *>(dev.wfrag);
    a.uoff = static_cast<const int *>(dev.uoff);
    a.choff = t.phased ? static_cast<const int *>(dev.choff) : nullptr;
    a.rowptr = static_cast<const int *>(direct.rowptr);
    a.trip = static_cast<const uint32_t *>(direct.trip);
    // with several parts the kernel stores partial sums into the workspace `out` points to, and the reduction that follows
    // applies the epilogue
    a.bias = t.splits == 1 ? ep.bias : nullptr;
    a.relu = ep.relu && t.splits == 1 ? 1 : 0;
    a.splits = t.splits;
    a.blk_split = (t.nblk + t.splits - 1) / t.splits;
    a.split_stride = t.splits > 1 ? split_stride : 0;
    a.short_rows = dev.short_rows ? 1 : 0;
    if (t.splits < 1 || (t.splits - 1) * a.blk_split >= t.nblk) return SCONV_ERR_PLAN; // a part without blocks
    const int64_t HW = (int64_t)d.H * d.W, P = (int64_t)N * g.OH * g.OW;
    if (!mfma_fits(d, N, feature_major)) return SCONV_ERR_RANGE;
    a.P = (int)P; a.OHW = g.OH * g.OW; a.OW = g.OW; a.OH = g.OH; a.H = d.H; a.W = d.W; a.Kg = g.Kg;
    a.pad = d.pad; a.stride = d.stride;
    a.cstep = t.cstep; a.lstep = t.lstep; a.Rr = t.Rr; a.Wl = t.Wl; a.row_img = (g.OH - 1) * t.lstep + t.Rr;
    a.g8 = t.g8; a.nblk = t.nblk; a.steps = t.steps; a.steps_last = t.steps_last; a.total_steps = t.total_steps;
    a.c_virtual = t.c_virtual;
    a.plane = t.plane;
    const int bn = 128 * t.nt;
    a.n_ptiles = (int)((P + bn - 1) / bn);
    a.n_mtiles = t.n_mtiles;
    a.n_tiles32 = t.n_tiles32;
    a.groups = d.groups;
    if (feature_major) {
        a.in_ch4 = N * 4; a.in_img = 1; a.in_group = 0; a.in_floats = (int64_t)d.C * N;
        a.out_img = 1; a.out_row = N; a.goff_mul = N;
    } else {
        a.in_ch4 = (int)(HW * 4); a.in_img = d.C * HW; a.in_group = g.Cg * HW; a.in_floats = (int64_t)N * d.C * HW;
        a.out_img = (int64_t)d.K * a.OHW; a.out_row = a.OHW; a.goff_mul = 1;
    }
    a.quads = (d.W + 3) / 4;
    // (a four's table entry has 8 bytes, a cell's 4: a row's fours need no more room)
    a.wide = t.cstep == 1 && d.W >= 4 && t.Wl >= d.W + d.pad && 2 * a.quads <= t.Wl;
    a.d_quads = make_fastdiv(a.quads, 1024);
    // what the kernel assumes
    if (t.plane > 1024 || t.total_steps > (1 << 18) || (int64_t)t.g8 * t.plane * 48 + 8 * (t.steps + t.steps_last) + 4 * t.plane > t.lds_bytes || t.g8 > 16 || t.nt > t.nt_max) return SCONV_ERR_PLAN;
    const int units = a.n_mtiles * d.groups * t.splits;
    const int64_t grid = (int64_t)a.n_ptiles * units;
    if (grid > 0x7fffffff) return SCONV_ERR_RANGE;
    a.d_units = make_fastdiv(units, std::max<int64_t>(grid / 8, 8 * (int64_t)units));
    a.d_splits = make_fastdiv(t.splits, units);
    a.d_mt = make_fastdiv(a.n_mtiles, units);
    a.d_ohw = make_fastdiv(a.OHW, P + bn);
    a.d_ow = make_fastdiv(a.OW, a.OHW);
    a.d_wl = make_fastdiv(a.Wl, 1025);
    a.d_rowimg = make_fastdiv(a.row_img, 1024);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (t.column && (!t.one_tap || t.nt != 1 || (t.nblk > 1 && t.g8 % 2) || t.mt > t.n_tiles32)) return SCONV_ERR_PLAN;
#define X(M, NN) \
    if (t.mt == M && t.nt == NN) \
        return launch_mfma_inst(!t.column ? sconv_mfma_kernel<M, NN> : a.c_virtual % 16 ? sconv_mfma_column_kernel<M, true> : sconv_mfma_column_kernel<M, false>, \
                                a, (int)grid, t.lds_bytes, s, hip_err);
    X(1, 1) X(2, 1)
#undef X
#define X(M, NN) if (t.mt == M && t.nt == NN) return launch_mfma_inst(sconv_mfma_kernel<M, NN>, a, (int)grid, t.lds_bytes, s, hip_err);
    X(1, 2) X(2, 2)
#undef X
    return SCONV_ERR_PLAN;
}

} // namespace sconv
