// Flat streams on the matrix cores: convolutions whose rows are long enough (SCONV_MC_ROW and the lines after it).
//
// v_smfmac_f32_16x16x64_f16 multiplies 16 filters by 64 columns of which each filter keeps two of every four: at a density of
// 0.1 four neighbouring channels hold more than two weights of a row in 0.4 % of the cases, so the zeros cost half of what they
// cost a dense product, and the rate is twice the dense one.  Measured in a loop without memory: 3.37 POP/s with random
// operands, 4.6 with zeros (the clock falls to 1.65 GHz under this load); 32x32x32 3.0.  A matrix step takes eight channel
// octets, each any octet at any filter tap: a lane reads the 16 bytes of an octet at its position, so a tap is an LDS address.
// Where a row has three or four of four channels the octet comes a second time, for all tiles of a wave or, if few tiles need
// it, in a step in which every tile has octets of its own (four times the LDS reads: 2 us where a shared step takes 1.1).
//
// Numbers: an fp32 value is h + l / 2^11, both fp16, at one power of two for a workgroup's activations and one for the weights;
// of 24 significant bits 23 or 24 remain.  h*h goes to one accumulator, l*h + h*l to a second one, l*l is left out: up to 2^-22
// of a product, 2^-24.6 as the mean square goes.  l is kept 2^11 larger than its value: at a value 2^27 below the largest fp16 the
// split still loses nothing, and 2^-18 of the value at 2^33 below.  The scale is taken from the first activations a workgroup
// stages: their largest goes to 2^12.  Where a later block holds one from 2^15 on, the scale and the sums shrink and the block is
// staged again.  Smaller ones that matter (`small_sum`), infinities and NaN send the workgroup back (`again`): one pass for every
// window of 26 binades that occurs, each at its own scale, and a pass that counts which stored weights meet an infinity.
// What that costs, 13x13, 256 -> 384, batch 256 (ordinary inputs 140-155 us in that run, the vector kernel 160-190): channels of
// magnitudes e^1 apart (sigma of the logarithm) 149, lognormal activations (sigma 2) 166, later channels 100 times the first ones
// 167, an outlier of 60 sigma an image 140; channels e^2 apart 365, every other image 2^-28 695, an outlier of 1e4 sigma or an
// infinity an image 710, a single infinity 293, magnitudes 1e-20 to 1e20 1840.
//
// Sums: the matrix instruction truncates small products against a large sum.  Up to 48 x 64 or 64 x 32 a wave there are registers
// for totals: every six steps the large accumulator is added to one, and keeps what that addition rounds off.  (384 -> 384, density
// 0.5, against plain additions every four steps, and the error at 800 nonzeros in 1e-8: every four 3.6 % slower, 11.0; every six
// 1.9 %, 11.8; every eight 0.7 %, 12.9; plain ones 13.0.)
// Error against 64 bits, relative 2-norm in 1e-8, of a row of n nonzeros on rectified normals, totals / none / fp32 chain /
// three-part kernel (sconv_mfma.hip): n = 60 9.4 / 11.9 / 9.9 / -, 120 9.9 / 14.3 / 13.7 / 5.5, 346 11 / 21 / 23 / 8.6, 800 12.0 /
// 27 / 35 / 12.9, 2304 13 / 32 / 62 / 23.  A call comes here where no row is off by more than on the kernel that it leaves: the lines
// in sconv_internal.h.
//
// A workgroup is four waves, 16 * mt filters x 16 * nt positions each, two along the filters or one; it walks the channels in
// blocks staged as [octet][row][high, low part][cell] of 16-byte units.  The pitch of a row is the number of positions in an
// output row modulo 16: sixteen lanes that run over the end of a row then still hit all banks; an octet is a multiple of 16 units,
// since lanes of two quarters are served together (conflicts 46 % of the LDS cycles with rows back to back, 25 % now: what is
// left are steps whose octets lie at different taps).  Activations are loaded four neighbouring cells x 8 channels a lane: the address unit takes
// 16 clocks an instruction, and one cell a lane kept it busy for 5 of the 8 us that staging a block took.  Weights go from L2 to
// registers, a step ahead.  Results leave through LDS, four positions a lane: 16 positions x 4 rows an instruction took 19 us
// for what takes 5.5.
//
// Measured, vector kernel -> here: 13x13, 256 -> 384, 3x3, batch 256, density 0.1: 160 -> 134 us; 28x28, 192 -> 128, 3x3, batch
// 64, density 0.2: 120 -> 66; 227x227, 3 -> 96, 11x11 stride 4, batch 64, density 0.3: 111 -> 93; three-part kernel -> here: 13x13,
// 384 -> 384 in two groups, batch 256, density 0.5: 251 -> 206.  439 random layers that the model sends here: 1.28x, from 0.83 to 3.1
// (the factors in sconv_api.cpp keep the lowest away).
// The first (time stamps, profiles/sconv_flat_mc_kernel.txt): of a workgroup's 73 us 38 are its 39 shared steps, 1570 clocks each for
// the 1536 of matrix instructions of the two waves on a SIMD, at 1.6 GHz (spilled registers had made it 2010); 7 private steps, 17
// staging, 5 before the first load, 7 the end and the stores.  With activations of all zero bits it took 133 us for 148.  Two
// workgroups out of step by half a block: no faster; one workgroup of 512 registers a lane and 128 positions a wave: 169 us; the next
// block's loads in flight across the last step: spills, 390 us.
#include <algorithm>
#include <type_traits>

#include "sconv_device.h"
#include "sconv_mc_walk.h"

namespace sconv {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef short s16x8v __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
using const_u32 = const __attribute__((address_space(4))) unsigned;
using const_i32 = const __attribute__((address_space(4))) int;

__device__ float mc_buffer_load(int4v rsrc, int voffset, int soffset, int aux) __asm("llvm.amdgcn.raw.buffer.load.f32");
typedef int int3v __attribute__((ext_vector_type(3)));
typedef int int2v __attribute__((ext_vector_type(2)));
__device__ int2v mc_buffer_load2(int4v rsrc, int voffset, int soffset, int aux) __asm("llvm.amdgcn.raw.buffer.load.v2i32");
__device__ int3v mc_buffer_load3(int4v rsrc, int voffset, int soffset, int aux) __asm("llvm.amdgcn.raw.buffer.load.v3i32");
__device__ int4v mc_buffer_load4(int4v rsrc, int voffset, int soffset, int aux) __asm("llvm.amdgcn.raw.buffer.load.v4i32");

#define INLINE __attribute__((always_inline))

struct FlatMcArgs {
    const float *in;
    float *out;
    const char *stream;      // records, see SCONV_MC_RECORD
    const int2 *seg;         // [group][unit][block]: first record, shared steps | private steps << 16
    const int *row_of;       // [group][unit][16 * mt]: output channel or -1
    const int *choff;        // phase form: byte offset of a virtual channel relative to its group, else null
    const float *bias;
    int relu;
    int P, OHW, OW, OH, H, W, pad;
    int cstep, lstep;        // input elements per cell; cells per output position
    int Rr, Wl, row_img;     // filter rows in cells, cells per staged row, staged rows of a whole image
    int g8, nblk, c_virtual;
    int plane;               // cells that are staged at most, a multiple of 64
    int run_until;           // phase form with runs: first position of the first workgroup whose fours of columns may pass the input's end
    int wide;                // four neighbouring cells are 16 consecutive bytes of the input: 1 along rows, 2 along the positions
    int quads;               // wide = 1: fours of cells per row, the last one back by what it would pass the row's end
    int pitch, part, octet;  // 16-byte units of LDS from one row of cells, high to low part, one channel octet to the next
    int words_at;            // four words of LDS behind the staged block, its table and the results
    int n_ptiles, n_mtiles, groups, n_units;
    int wr;                  // waves along the filters: 2 (then 2 along the positions) or 1 (then 4)
    int splits, blk_split;   // workgroups along the channel blocks, blocks each of them takes
    long long split_stride;  // floats from one part's sums to the next (out then is the workspace)
    int in_ch4;              // bytes from one channel to the next
    long long in_img, in_group;   // floats from one image / one group's channels to the next
    long long in_floats;     // floats of the whole input
    long long stream_bytes;
    long long out_img, out_row;
    int wexp;                // weights are packed times 2^wexp
    float small_sum;         // sums below it may be of activations that all have lost bits
    FastDiv d_units, d_splits, d_mt, d_ohw, d_ow, d_wl, d_rowimg, d_quads;
};

#define SCONV_MAGIC(D) 0xffffffffu / D + 1u
static __constant__ unsigned kMcPieceMagic[17] = {0, 0, SCONV_MAGIC(2), SCONV_MAGIC(3), SCONV_MAGIC(4), SCONV_MAGIC(5), SCONV_MAGIC(6), SCONV_MAGIC(7),
    SCONV_MAGIC(8), SCONV_MAGIC(9), SCONV_MAGIC(10), SCONV_MAGIC(11), SCONV_MAGIC(12), SCONV_MAGIC(13), SCONV_MAGIC(14), SCONV_MAGIC(15), SCONV_MAGIC(16)};
#undef SCONV_MAGIC

// x * scale = h + l / 2^11, both fp16
static __device__ __forceinline__ void split8_f16(const float (&x)[8], float scale, uint4 &h, uint4 &l)
{
    unsigned hw[4], lw[4];
    const float scale_l = scale * 2048.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const f32x2 v = {x[2 * i] * scale, x[2 * i + 1] * scale};
        const f16x2 hb = __builtin_convertvector(v, f16x2);
        // (exact: the difference has no more bits than x)
        const f32x2 r = {__builtin_fmaf((float)hb[0], -2048.f, x[2 * i] * scale_l), __builtin_fmaf((float)hb[1], -2048.f, x[2 * i + 1] * scale_l)};
        const f16x2 lb = __builtin_convertvector(r, f16x2);
        hw[i] = __builtin_bit_cast(unsigned, hb);
        lw[i] = __builtin_bit_cast(unsigned, lb);
    }
    h = make_uint4(hw[0], hw[1], hw[2], hw[3]);
    l = make_uint4(lw[0], lw[1], lw[2], lw[3]);
}

static __device__ __forceinline__ bool mc_not_finite(float v) { return (__float_as_uint(v) & 0x7f800000u) == 0x7f800000u; }

// The infinities and NaN among eight activations: 1 in h where a positive one is (a NaN is both), 1 in l where a negative one
static __device__ __forceinline__ void marks8_f16(const float (&x)[8], uint4 &h, uint4 &l)
{
    unsigned hw[4], lw[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        hw[i] = lw[i] = 0;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const float v = x[2 * i + e];
            if (v == __builtin_inff() || v != v) hw[i] |= 0x3c00u << (16 * e);
            if (v == -__builtin_inff() || v != v) lw[i] |= 0x3c00u << (16 * e);
        }
    }
    h = make_uint4(hw[0], hw[1], hw[2], hw[3]);
    l = make_uint4(lw[0], lw[1], lw[2], lw[3]);
}

struct McTile {
    int ptile, split, g, mt;
};
static __device__ __forceinline__ McTile mc_tile_of(const FlatMcArgs &a, int bid)
{
    const int units = a.n_mtiles * a.groups * a.splits, full = (a.n_ptiles >> 3) * 8 * units;
    McTile t;
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

// again = false: a workgroup's sums, stored with the epilogue; true if they have to be taken again.
// again = true: those sums once more, a window of magnitudes after the other.
template <int MT, int NT, bool again>
static __device__ __forceinline__ bool mc_tile(const FlatMcArgs &a, int bid, char *lds)
{
    constexpr int kBatch = 4, kRec = SCONV_MC_RECORD(MT), kIdx = (MT + 1) / 2;
    static_assert(MT >= 2 && MT <= 4, "");
    const int lane = threadIdx.x & 63, quarter = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const McTile tile = mc_tile_of(a, bid);
    const int g = tile.g;
    const int b_first = tile.split * a.blk_split, b_end = min(b_first + a.blk_split, a.nblk);   // this workgroup's channel blocks
    const int unit = g * a.n_units + tile.mt * a.wr + (a.wr == 2 ? wave >> 1 : 0), pwave = a.wr == 2 ? wave & 1 : wave;
    const int bn = 16 * NT * (a.wr == 2 ? 2 : 4);

    const int p0 = tile.ptile * bn;
    const int n_first = fdiv(p0, a.d_ohw), y_first = fdiv(p0 - n_first * a.OHW, a.d_ow);
    const int rows_first = (a.OH - 1 - y_first) * a.lstep + a.Rr;      // staged rows of the first image
    auto row_at = [&](int n, int y) {
        return n == n_first ? (y - y_first) * a.lstep : rows_first + (n - n_first - 1) * a.row_img + y * a.lstep;
    };
    int cells;
    {
        const int p1 = min(p0 + bn, a.P) - 1;
        const int n = fdiv(p1, a.d_ohw), y = fdiv(p1 - n * a.OHW, a.d_ow);
        cells = (row_at(n, y) + a.Rr) * a.Wl;
    }
    const unsigned part16 = (unsigned)a.part * 16u;
    unsigned lane_addr[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int p = min(p0 + (pwave * NT + t) * 16 + (lane & 15), a.P - 1);
        const int n = fdiv(p, a.d_ohw), q = p - n * a.OHW, y = fdiv(q, a.d_ow), x = q - y * a.OW;
        lane_addr[t] = (unsigned)(row_at(n, y) * a.pitch + x * a.lstep) * 16u;
    }
    // where the cells come from, relative to image n_first, and where they go in LDS (a table behind the staged block): padding and
    // cells past the end read beyond the buffer.  What no cell is written to stays zero: the right padding of a row.
    const int block16 = a.g8 * a.octet;
    uint2 *table = reinterpret_cast<uint2 *>(lds + (size_t)block16 * 16);
    // the largest of the first activations; flags, read while other waves already store their results
    unsigned *word = reinterpret_cast<unsigned *>(lds + a.words_at);
    for (int i = threadIdx.x; i < block16; i += 256) reinterpret_cast<uint4 *>(lds)[i] = make_uint4(0, 0, 0, 0);
    const bool wide = !again && a.wide;
    const int n_rows = fdiv(cells, a.d_wl), n_quads = !wide ? 0 : a.wide == 1 ? n_rows * a.quads : cells >> 2;
    for (int i = threadIdx.x; i < (wide ? n_quads : a.plane); i += 256) {
        int row, col;            // of the cell, or of the first of four
        if (wide && a.wide == 1) {
            row = fdiv(i, a.d_quads);
            col = a.pad + min((i - row * a.quads) * 4, a.W - 4);
        } else {
            const int cell = wide ? i * 4 : i;
            row = fdiv(cell, a.d_wl);
            col = cell - row * a.Wl;
        }
        int n = 0, yp = y_first * a.lstep + row;
        if (row >= rows_first) {
            const int img = fdiv(row - rows_first, a.d_rowimg);
            n = 1 + img;
            yp = row - rows_first - img * a.row_img;
        }
        const int iy = yp * a.cstep - a.pad, ix = col * a.cstep - a.pad;
        const bool there = wide || i < cells, ok = there && iy >= 0 && iy < a.H && ix >= 0 && ix < a.W;
        // (fours of a padding row stay as they are, zero)
        table[i] = make_uint2(ok ? (unsigned)(n * (int)a.in_img + iy * a.W + ix) * 4u : 0x80000000u,
                              there && (ok || !wide) ? (unsigned)(row * a.pitch + col) * 16u : 0xffffffffu);
    }
    const FastDiv d_nquads = {(unsigned)n_quads, n_quads > 1 ? 0xffffffffu / (unsigned)n_quads + 1u : 0u};
    if (threadIdx.x == 0) word[0] = word[1] = word[2] = word[3] = 0;
    const int pieces = (cells + 63) >> 6;
    const FastDiv d_pieces = {(unsigned)pieces, ((const_u32 *)kMcPieceMagic)[pieces]};
    int4v rsrc;
    {
        const float *src = a.in + n_first * a.in_img + g * a.in_group;
        const unsigned long long ip = (unsigned long long)src;
        const long long left = (a.in_floats - (n_first * a.in_img + g * a.in_group)) * 4;
        rsrc.x = __builtin_amdgcn_readfirstlane((int)(unsigned)ip);
        rsrc.y = __builtin_amdgcn_readfirstlane((int)(unsigned)(ip >> 32));
        rsrc.z = __builtin_amdgcn_readfirstlane((int)min(left, 0x7fffffffll));
        rsrc.w = 0x00020000;
    }
    // weights: record by record from a scalar offset, the record of the next step on its way while one is multiplied (the stream
    // ends with a spare record)
    const_i32 *seg = (const_i32 *)(a.seg + (size_t)unit * a.nblk);
    int4v wrsrc;
    {
        const long long first = (long long)seg[2 * b_first] * kRec;
        const unsigned long long wp = (unsigned long long)(a.stream + first);
        wrsrc.x = __builtin_amdgcn_readfirstlane((int)(unsigned)wp);
        wrsrc.y = __builtin_amdgcn_readfirstlane((int)(unsigned)(wp >> 32));
        wrsrc.z = __builtin_amdgcn_readfirstlane((int)min(a.stream_bytes - first, 0x7fffffffll));
        wrsrc.w = 0x00020000;
    }
    const int lane16 = lane * 16, meta = lane * (kIdx * 4 + 4);
    int wpos = 0;
    struct Record {
        f16x8 h[MT], l[MT];
        int idx[kIdx];
        int off;         // LDS address / 16 of this lane's two octets, the first | the second << 16; in private steps lane i of four has tile i's
    };
    auto load_record = [&](Record &r) INLINE {
        if constexpr (kIdx == 2) {
            const int3v o = mc_buffer_load3(wrsrc, meta, wpos + MT * 2048, 0);
            r.idx[0] = o.x; r.idx[1] = o.y; r.off = o.z;
        } else {
            const int2v o = mc_buffer_load2(wrsrc, meta, wpos + MT * 2048, 0);
            r.idx[0] = o.x; r.off = o.y;
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            r.h[m] = __builtin_bit_cast(f16x8, mc_buffer_load4(wrsrc, lane16, wpos + m * 2048, 0));
            r.l[m] = __builtin_bit_cast(f16x8, mc_buffer_load4(wrsrc, lane16 + 1024, wpos + m * 2048, 0));
        }
        wpos += kRec;
    };
    // the record that stands at the beginning of block b
    auto first_record = [&](Record &r, int b) INLINE {
        wpos = mc_block_at(seg, b, b_first, kRec);
        load_record(r);
    };
    auto offset_of = [&](int off, int m) INLINE {   // tile m's of a private step
        return m == 0 ? __builtin_amdgcn_mov_dpp(off, 0x00, 0xf, 0xf, true) : m == 1 ? __builtin_amdgcn_mov_dpp(off, 0x55, 0xf, 0xf, true) :
               m == 2 ? __builtin_amdgcn_mov_dpp(off, 0xaa, 0xf, 0xf, true) : __builtin_amdgcn_mov_dpp(off, 0xff, 0xf, 0xf, true);
    };
    struct Cols {
        f16x16 h, l;
    };
    auto load_cols = [&](Cols &b, int t, int off) INLINE {
        const char *p0 = lds + lane_addr[t] + ((unsigned)off & 0xffffu) * 16u, *p1 = lds + lane_addr[t] + ((unsigned)off >> 16) * 16u;
        const f16x8 h0 = *reinterpret_cast<const f16x8 *>(p0), h1 = *reinterpret_cast<const f16x8 *>(p1);
        const f16x8 l0 = *reinterpret_cast<const f16x8 *>(p0 + part16), l1 = *reinterpret_cast<const f16x8 *>(p1 + part16);
        b.h = __builtin_shufflevector(h0, h1, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
        b.l = __builtin_shufflevector(l0, l1, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
    };

    constexpr bool kTotals = SCONV_MC_TOTALS(MT, NT);
    f32x4 acc[MT][NT], cor[MT][NT], tot[kTotals ? MT : 1][kTotals ? NT : 1];
    auto clear = [&]() INLINE {
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                acc[m][t] = cor[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (kTotals) tot[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
    };
    // (What the total's rounding leaves out stays in the accumulator.  In this order both are changed in place: with the sum in a
    // variable of its own a second set of totals is live, 117 spilled registers with 48 x 64 a wave.)
    auto flush = [&]() INLINE {
        if constexpr (kTotals)
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const f32x4 grown = (tot[m][t] + acc[m][t]) - tot[m][t];
                    acc[m][t] -= grown;
                    tot[m][t] += grown;
                }
    };
    auto sum_of = [&](int m, int t, int r) INLINE {
        const float v = __builtin_fmaf(cor[m][t][r], 0x1p-11f, acc[m][t][r]);
        if constexpr (kTotals) return tot[m][t][r] + v;
        else return v;
    };
#define SCONV_SMFMAC(D, M, T, A, B, I) \
    D[M][T] = (M) & 1 ? __builtin_amdgcn_smfmac_f32_16x16x64_f16(A, B, D[M][T], I, 0, 1) : __builtin_amdgcn_smfmac_f32_16x16x64_f16(A, B, D[M][T], I, 0, 0)
    auto multiply = [&](const Record &r, const Cols &b, int t, int m0, int m1) INLINE {
#pragma unroll
        for (int m = m0; m < m1; ++m) SCONV_SMFMAC(acc, m, t, r.h[m], b.h, r.idx[m >> 1]);
#pragma unroll
        for (int m = m0; m < m1; ++m) SCONV_SMFMAC(cor, m, t, r.l[m], b.h, r.idx[m >> 1]);
#pragma unroll
        for (int m = m0; m < m1; ++m) SCONV_SMFMAC(cor, m, t, r.h[m], b.l, r.idx[m >> 1]);
    };
    // stored weights on infinities: acc counts products that are +infinity, cor those that are -infinity (a stored zero, -0
    // here, makes NaN of either and counts as both)
    auto count = [&](const Record &r, const Cols &b, int t, int m0, int m1) INLINE {
#pragma unroll
        for (int m = m0; m < m1; ++m) {
            const s16x8v w = __builtin_bit_cast(s16x8v, r.h[m]);
            const f16x8 up = __builtin_bit_cast(f16x8, (s16x8v)(((w > 0) | (w == (short)0x8000)) & (short)0x3c00));
            const f16x8 down = __builtin_bit_cast(f16x8, (s16x8v)((w < 0) & (short)0x3c00));
            SCONV_SMFMAC(acc, m, t, up, b.h, r.idx[m >> 1]);
            SCONV_SMFMAC(acc, m, t, down, b.l, r.idx[m >> 1]);
            SCONV_SMFMAC(cor, m, t, down, b.h, r.idx[m >> 1]);
            SCONV_SMFMAC(cor, m, t, up, b.l, r.idx[m >> 1]);
        }
    };
#undef SCONV_SMFMAC
    const_i32 *choff = (const_i32 *)a.choff;

    // items of 64 cells x 8 channels are dealt to the waves; the loads of up to kBatch of them are in flight together
    struct Batch {
        float x[kBatch][8];
    };
    auto load_items = [&](Batch &v, int b, int i0, int items) INLINE {
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const int item = min(i0 + 4 * j, items - 1), o = fdiv(item, d_pieces), piece = item - o * pieces, c = b * a.g8 * 8 + o * 8;
            const unsigned vo = i0 + 4 * j < items ? table[piece * 64 + lane].x : 0x80000000u;
            // Phases of a stride of 4 or 8: four channels a load, side by side in the input.  One a load and 16 bytes from lane to lane
            // the address unit saw four times the instructions and every line four times: 3 -> 96, 227x227, 11x11 stride 4, batch
            // 64: 94 -> 88 us.
            if (p0 < a.run_until) {
#pragma unroll
                for (int i = 0; i < 8; i += 4) {
                    const int co = choff[c + i];
                    const f32x4 r = __builtin_bit_cast(f32x4, mc_buffer_load4(rsrc, (int)(vo | ((unsigned)co & 0x80000000u)), co & 0x7fffffff, 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e) v.x[j][i + e] = r[e];
                }
                continue;
            }
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
                v.x[j][i] = mc_buffer_load(rsrc, (int)(vo | ((unsigned)co[i] & 0x80000000u)), co[i] & 0x7fffffff, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto store_item = [&](int item, const uint4 &h, const uint4 &l) INLINE {
        const int o = fdiv(item, d_pieces), piece = item - o * pieces;
        const unsigned at = table[piece * 64 + lane].y;
        if (at == 0xffffffffu) return;
        char *dst = lds + (size_t)o * a.octet * 16 + at;
        *reinterpret_cast<uint4 *>(dst) = h;
        *reinterpret_cast<uint4 *>(dst + part16) = l;
    };
    auto items_of = [&](int b) { return min(a.g8, (a.c_virtual - b * a.g8 * 8 + 7) >> 3) * pieces; };

    // f(output, row, the sum, its two accumulators) for every output of this lane
    auto outputs = [&](auto f) INLINE {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int p = p0 + (pwave * NT + t) * 16 + (lane & 15);
            if (p >= a.P) continue;
            const int n = fdiv(p, a.d_ohw);
            float *dst = a.out + tile.split * a.split_stride + n * a.out_img + (p - n * a.OHW);
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const int4v rows = *reinterpret_cast<const int4v *>(a.row_of + (size_t)unit * (16 * MT) + m * 16 + quarter * 4);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int k = r == 0 ? rows.x : r == 1 ? rows.y : r == 2 ? rows.z : rows.w;
                    if (k < 0) continue;
                    f(dst[k * a.out_row], k, sum_of(m, t, r), acc[m][t][r], cor[m][t][r]);
                }
            }
        }
    };

    if constexpr (!again) {
        clear();
        Record r0;
        float scale = 1.f;
        int expo = 0;                        // activations are staged times 2^expo
        unsigned least = 0xffffffffu;        // smallest nonzero magnitude, twice its bits less one
        // (the largest so far goes to [2^12, 2^13))
        auto largest = [&]() INLINE { return (int)(__builtin_amdgcn_readfirstlane(*(volatile unsigned *)word) >> 23); };
        auto set_scale = [&](int e) INLINE {
            expo = 139 - (e == 0 ? 129 : max(e, 40));
            scale = __uint_as_float((unsigned)(127 + expo) << 23);
        };
        auto magnitude = [&](float v) INLINE {
            const unsigned u = __float_as_uint(v) & 0x7fffffffu;
            return u < 0x7f800000u ? u : 0u;
        };
        float most = 0.f;                    // largest magnitude of a block, infinities among them
        auto note = [&](float v0, float v1) INLINE {
            least = min(least, min((__float_as_uint(v0) << 1) - 1u, (__float_as_uint(v1) << 1) - 1u));
            asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(most) : "v"(v0), "v"(v1));   // (fmaxf would quiet every loaded value first)
        };
        // wide: items of 64 lanes, four cells x 8 channels each, counted through a block's octets
        struct Four {
            f32x4 x[8];
            unsigned at;
        };
        auto fours_of = [&](int b) { return min(a.g8, (a.c_virtual - b * a.g8 * 8 + 7) >> 3) * n_quads; };
        auto load_fours = [&](Four &v, int b, int i0) INLINE {
            const int fours = fours_of(b), i = i0 + lane, o = fdiv(min(i, fours - 1), d_nquads);
            const uint2 e = table[min(i, fours - 1) - o * n_quads];
            const int c = (b * a.g8 + o) * 8;
            v.at = i < fours && e.y != 0xffffffffu ? e.y + (unsigned)(o * a.octet) * 16u : 0xffffffffu;
            const unsigned vo = i < fours ? e.x + (unsigned)(c * a.in_ch4) : 0x80000000u;
#pragma unroll
            for (int q = 0; q < 8; ++q)
                v.x[q] = __builtin_bit_cast(f32x4, mc_buffer_load4(rsrc, (int)(c + q < a.c_virtual ? vo + (unsigned)(q * a.in_ch4) : 0x80000000u), 0, 0));
            __builtin_amdgcn_sched_barrier(0);
        };
        auto split_fours = [&](const Four &v) INLINE {
            if (v.at != 0xffffffffu) {
                char *dst = lds + v.at;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x[8] = {v.x[0][e], v.x[1][e], v.x[2][e], v.x[3][e], v.x[4][e], v.x[5][e], v.x[6][e], v.x[7][e]};
#pragma unroll
                    for (int q = 0; q < 8; q += 2) note(x[q], x[q + 1]);
                    uint4 h, l;
                    split8_f16(x, scale, h, l);
                    *reinterpret_cast<uint4 *>(dst + e * 16) = h;
                    *reinterpret_cast<uint4 *>(dst + e * 16 + part16) = l;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        __syncthreads();                     // the table is there
        bool unscaled = true;
        int since = 0;                       // steps since the totals were added to
        for (int b = b_first; b < b_end;) {
            most = 0.f;
            if (wide) {
                const int fours = fours_of(b);
                int i0 = wave * 64;
                Four v0, v1;
                load_fours(v0, b, i0);
                if (unscaled) {
                    unsigned first = 0;
#pragma unroll
                    for (int q = 0; q < 8; ++q)
#pragma unroll
                        for (int e = 0; e < 4; ++e) first = max(first, magnitude(v0.x[q][e]));
                    if (first) atomicMax(word, first);
                    __syncthreads();
                    set_scale(largest());
                } else {
                    __syncthreads();         // the block before is used up
                }
                for (;;) {
                    if (i0 + 256 >= fours) break;
                    load_fours(v1, b, i0 + 256);
                    split_fours(v0);
                    i0 += 256;
                    if (i0 + 256 >= fours) {
                        v0 = v1;
                        break;
                    }
                    load_fours(v0, b, i0 + 256);
                    split_fours(v1);
                    i0 += 256;
                }
                first_record(r0, b);
                split_fours(v0);
            } else {
                const int items = items_of(b);
                Batch y0, y1;
                auto split_items = [&](Batch &v, int i0) INLINE {
#pragma unroll
                    for (int j = 0; j < kBatch; ++j) {
                        const int item = i0 + 4 * j;
                        if (item >= items) break;
#pragma unroll
                        for (int i = 0; i < 8; i += 2) note(v.x[j][i], v.x[j][i + 1]);
                        uint4 h, l;
                        split8_f16(v.x[j], scale, h, l);
                        store_item(item, h, l);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                };
                int i0 = wave;
                load_items(y0, b, i0, items);
                if (unscaled) {
                    unsigned first = 0;
#pragma unroll
                    for (int j = 0; j < kBatch; ++j)
#pragma unroll
                        for (int i = 0; i < 8; ++i) first = max(first, magnitude(y0.x[j][i]));
                    if (first) atomicMax(word, first);
                    __syncthreads();
                    set_scale(largest());
                } else {
                    __syncthreads();
                }
                for (;;) {
                    if (i0 + 4 * kBatch >= items) break;
                    load_items(y1, b, i0 + 4 * kBatch, items);
                    split_items(y0, i0);
                    i0 += 4 * kBatch;
                    if (i0 + 4 * kBatch >= items) {
                        y0 = y1;
                        break;
                    }
                    load_items(y0, b, i0 + 4 * kBatch, items);
                    split_items(y1, i0);
                    i0 += 4 * kBatch;
                }
                first_record(r0, b);
                split_items(y0, i0);
            }
            // From 2^15 on a value is too large for the scale: it shrinks, with what is summed, and the block is staged again.
            // (A loop that runs once: with a branch the compiler keeps a second set of accumulators, 200 spilled registers.)
            if (most >= __uint_as_float((unsigned)min(142 - expo, 255) << 23) && most < __builtin_inff()) atomicMax(word, __float_as_uint(most));
            __syncthreads();
            unscaled = false;
            const bool over = largest() > 141 - expo;
            for (int k = over; k; --k) {
                const int before = expo;
                set_scale(largest());
                const float down = __builtin_ldexpf(1.f, expo - before);
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                    {
                        acc[m][t] *= down;
                        cor[m][t] *= down;
                        if constexpr (kTotals) tot[m][t] *= down;
                    }
            }
            const unsigned steps = over ? 0u : (unsigned)seg[2 * b + 1];
            const int n_shared = (int)(steps & 0xffffu), n_private = (int)(steps >> 16);
            Cols c0, c1;
            auto shared_step = [&](const Record &cur, const Record &next) INLINE {
#pragma unroll
                for (int t = 0; t < NT; t += 2) {
                    load_cols(c1, t + 1, cur.off);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(cur, c0, t, 0, MT);
                    __builtin_amdgcn_sched_barrier(0);
                    if (t + 2 < NT) load_cols(c0, t + 2, cur.off);
                    else load_cols(c0, 0, next.off);   // (a private step's, or none: not used)
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(cur, c1, t + 1, 0, MT);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            auto private_step = [&](const Record &cur, const Record &) INLINE {
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    const int off = offset_of(cur.off, m);
                    load_cols(c0, 0, off);
#pragma unroll
                    for (int t = 0; t < NT; t += 2) {
                        load_cols(c1, t + 1, off);
                        __builtin_amdgcn_sched_barrier(0);
                        multiply(cur, c0, t, m, m + 1);
                        __builtin_amdgcn_sched_barrier(0);
                        if (t + 2 < NT) load_cols(c0, t + 2, off);
                        __builtin_amdgcn_sched_barrier(0);
                        multiply(cur, c1, t + 1, m, m + 1);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            };
            load_cols(c0, 0, r0.off);
            mc_walk_block(r0, n_shared, n_private, since, load_record, shared_step, private_step, [&](int left) INLINE {
                if (left || b + 1 < b_end) flush();          // (the last ones are added in sum_of)
            });
            b += !over;
        }
        // What the split did not carry: sums that are not finite, and sums that only small activations went into.  Scaled below
        // 2^-13 an activation has lost more than the two parts of a larger one lose (2^-23 of it), below 2^-35 it may be gone.
        // That counts where what goes into a sum is not much larger than what is lost, 2^-36.8 a product on average.  A sum may
        // be small by itself; the second accumulator, of the same size and no relation to it, is small as well only where all is.
        // (Ordinary inputs: one value in 3e7 of a normal distribution is below 2^-13, a workgroup stages 5e4 to 2e5 of them.  Sums
        // of 0, empty filters among them, count only where activations may be gone: with 2^-18 for that, 3 % of such calls took twice
        // as long.)
        volatile unsigned *const flag = word + 1;      // again; activations: byte 0 small, byte 1 gone; sums: byte 0 small, byte 1 small or 0
        volatile unsigned char *const lost = reinterpret_cast<volatile unsigned char *>(flag + 1), *const low = lost + 4;
        if (least < ((unsigned)(114 - expo) << 24) - 1u) lost[least < ((unsigned)max(92 - expo, 0) << 24) - 1u] = 1;
        bool bad = false;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    acc[m][t][r] = __builtin_ldexpf(sum_of(m, t, r), -(expo + a.wexp));
                    bad |= mc_not_finite(acc[m][t][r]);
                }
        if (bad) flag[0] = 1;
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(flag[1])) {
            unsigned smallest = 0xffffffffu;               // of the sums that are not zero, as `least`
            float smallest_or_0 = __builtin_inff();
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float v = fmaxf(fabsf(acc[m][t][r]), fabsf(__builtin_ldexpf(cor[m][t][r], -(expo + a.wexp))));
                        smallest = min(smallest, (__float_as_uint(v) << 1) - 1u);
                        smallest_or_0 = fminf(smallest_or_0, v);
                    }
            const float limit = __builtin_ldexpf(a.small_sum, -(expo + a.wexp));
            if (smallest < (__float_as_uint(limit) << 1)) low[0] = 1;
            if (smallest_or_0 < limit) low[1] = 1;
            __syncthreads();
        }
        if (flag[0] | (flag[1] & flag[2])) return true;
        // Through LDS, a wave's rows of 16 * NT positions each for itself: every store is whole rows of positions instead of 16.
        // (a pitch of 4 modulo 16 words: the 16 positions x 4 rows of a write fall into different banks)
        constexpr int kPos = 16 * NT, kPitch = kPos + 4, kRows = 64 / kPos;
        float *mine = reinterpret_cast<float *>(lds) + wave * (16 * MT * kPitch);
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) mine[(m * 16 + quarter * 4 + r) * kPitch + t * 16 + (lane & 15)] = acc[m][t][r];
        // a lane takes four positions of one row; a wave's row numbers and biases sit in its lanes
        const int per_row = kPos / 4, sub = lane / per_row, first = p0 + pwave * kPos + (lane & (per_row - 1)) * 4;
        const int my_row = 16 * MT < 64 && lane >= 16 * MT ? -1 : a.row_of[(size_t)unit * (16 * MT) + lane];
        const float my_bias = a.bias && my_row >= 0 ? a.bias[my_row] : 0.f;
        char *base = reinterpret_cast<char *>(a.out + tile.split * a.split_stride + n_first * a.out_img);
        unsigned at[4];
        bool valid[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int p = min(first + i, a.P - 1), n = fdiv(p, a.d_ohw);
            valid[i] = first + i < a.P;
            at[i] = (unsigned)((n - n_first) * (int)a.out_img + (p - n * a.OHW)) * 4u;
        }
        const bool whole = valid[3] && at[3] == at[0] + 12u;    // in one image: consecutive in memory
        const bool all_whole = __ballot(!whole) == 0ull;
        for (int r = sub; r < 16 * MT; r += 64 / per_row) {
            f32x4 v = *reinterpret_cast<const f32x4 *>(mine + r * kPitch + (lane & (per_row - 1)) * 4);
            const int k = __builtin_amdgcn_ds_bpermute(r * 4, my_row);
            const float bias = __uint_as_float((unsigned)__builtin_amdgcn_ds_bpermute(r * 4, (int)__float_as_uint(my_bias)));
            if (a.bias) v += bias;
            if (a.relu) v = f32x4{fmaxf(v[0], 0.f), fmaxf(v[1], 0.f), fmaxf(v[2], 0.f), fmaxf(v[3], 0.f)};
            char *dst = base + k * a.out_row * 4;
            if (k < 0) continue;
            if (all_whole) {
                *reinterpret_cast<f32x4u *>(dst + at[0]) = v;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (valid[i]) *reinterpret_cast<float *>(dst + at[i]) = v[i];
            }
        }
        return false;
    } else {
        // Which magnitudes there are: bit w for exponents 26 w .. 26 w + 25, bit 31 for infinities and NaN
        unsigned there = 0;
        __syncthreads();
        for (int b = b_first; b < b_end; ++b) {
            const int items = items_of(b);
            for (int i0 = wave; i0 < items; i0 += 4 * kBatch) {
                Batch v;
                load_items(v, b, i0, items);
#pragma unroll
                for (int j = 0; j < kBatch; ++j)
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const unsigned u = __float_as_uint(v.x[j][i]) & 0x7fffffffu;
                        if (u) there |= u >= 0x7f800000u ? 0x80000000u : 1u << ((u >> 23) / 26);
                    }
            }
        }
        if (there) atomicOr(word, there);
        __syncthreads();
        there = __builtin_amdgcn_readfirstlane(*(volatile unsigned *)word);
        // window 0 .. 9, or 31: infinities and NaN counted
        auto pass = [&](int window) INLINE {
            clear();
            wpos = 0;
            int since = 0;
            const float scale = __uint_as_float((unsigned)(242 - 26 * min(window, 9)) << 23);
            for (int b = b_first; b < b_end; ++b) {
                __syncthreads();
                const int items = items_of(b);
                for (int i0 = wave; i0 < items; i0 += 4 * kBatch) {
                    Batch v;
                    load_items(v, b, i0, items);
#pragma unroll
                    for (int j = 0; j < kBatch; ++j) {
                        const int item = i0 + 4 * j;
                        if (item >= items) break;
                        uint4 h, l;
                        if (window == 31) {
                            marks8_f16(v.x[j], h, l);
                        } else {
#pragma unroll
                            for (int i = 0; i < 8; ++i) {
                                const unsigned e = (__float_as_uint(v.x[j][i]) & 0x7fffffffu) >> 23;
                                v.x[j][i] = e < 255 && (int)(e / 26) == window ? v.x[j][i] : 0.f;
                            }
                            split8_f16(v.x[j], scale, h, l);
                        }
                        store_item(item, h, l);
                    }
                }
                __syncthreads();
                const unsigned steps = (unsigned)seg[2 * b + 1];
                const int n_shared = (int)(steps & 0xffffu), n_all = n_shared + (int)(steps >> 16);
                for (int i = 0; i < n_all; ++i) {
                    Record r;
                    Cols c;
                    load_record(r);
#pragma unroll
                    for (int m = 0; m < MT; ++m) {
                        const int off = i < n_shared ? r.off : offset_of(r.off, m);
#pragma unroll
                        for (int t = 0; t < NT; ++t) {
                            load_cols(c, t, off);
                            if (window == 31) count(r, c, t, m, m + 1);
                            else multiply(r, c, t, m, m + 1);
                        }
                    }
                    if (window != 31 && ++since == 6) {
                        flush();
                        since = 0;
                    }
                }
            }
        };
        // (through the output: there is no room for a second set of accumulators)
        outputs([&](float &out, int, float, float, float) INLINE { out = 0.f; });
        for (int w = 0; w < 10; ++w) {
            if (!(there >> w & 1)) continue;
            pass(w);
            outputs([&](float &out, int, float v, float, float) INLINE { out += __builtin_ldexpf(v, 26 * w - 115 - a.wexp); });
        }
        if (there >> 31) {
            pass(31);
            outputs([&](float &out, int, float, float up, float down) INLINE {
                if (up > 0.f) out += __builtin_inff();
                if (down > 0.f) out -= __builtin_inff();
            });
        }
        if (a.bias || a.relu)
            outputs([&](float &out, int k, float, float, float) INLINE {
                const float v = a.bias ? out + a.bias[k] : out;
                out = a.relu ? fmaxf(v, 0.f) : v;
            });
        return false;
    }
}

template <int MT, int NT>
__global__ void __launch_bounds__(256, 2) sconv_flat_mc_kernel(const FlatMcArgs a)
{
    extern __shared__ uint4 smem[];
    char *lds = reinterpret_cast<char *>(smem);
    if (!mc_tile<MT, NT, false>(a, blockIdx.x, lds)) return;
    // The rare rest reads the arguments again, out of the compiler's sight: with their values kept for it the first pass spills
    // scalar registers.
    unsigned long long args = (unsigned long long)__builtin_amdgcn_kernarg_segment_ptr();
    int bid = blockIdx.x;
    asm volatile("" : "+s"(args), "+s"(bid));
    const FlatMcArgs &b = *(const FlatMcArgs *)(const __attribute__((address_space(4))) FlatMcArgs *)args;
    __syncthreads();
    mc_tile<MT, NT, true>(b, bid, lds);
}

template <int MT, int NT>
static int launch_mc_inst(const FlatMcArgs &a, int grid, int lds_bytes, hipStream_t s, int *hip_err)
{
    auto kern = sconv_flat_mc_kernel<MT, NT>;
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

int launch_flat_mc(const sconv_desc &layer, const FlatMcTiling &t, const DeviceLds &dev, const float *in, float *out, int N,
                   const Epilogue &ep, int64_t split_stride, void *stream, int *hip_err)
{
    const sconv_desc d = mfma_desc(layer);
    const Geometry g = geometry(d);
    FlatMcArgs a;
    a.in = in;
    a.out = out;
    a.stream = static_cast<const char *>(dev.pairs);
    a.seg = static_cast<const int2 *>(dev.seg_ptr);
    a.row_of = static_cast<const int *>(dev.row_of);
    a.choff = t.phased ? static_cast<const int *>(dev.store_tbl) : nullptr;
    a.bias = t.splits == 1 ? ep.bias : nullptr;
    a.relu = ep.relu && t.splits == 1 ? 1 : 0;
    a.splits = t.splits;
    a.blk_split = (t.nblk + t.splits - 1) / t.splits;
    a.split_stride = t.splits > 1 ? split_stride : 0;
    if (t.splits < 1 || (t.splits - 1) * a.blk_split >= t.nblk) return SCONV_ERR_PLAN; // a part without blocks
    const int64_t HW = (int64_t)d.H * d.W, P = (int64_t)N * g.OH * g.OW;
    if (!mfma_fits(d, N, false)) return SCONV_ERR_RANGE;
    a.P = (int)P; a.OHW = g.OH * g.OW; a.OW = g.OW; a.OH = g.OH; a.H = d.H; a.W = d.W;
    a.pad = d.pad;
    a.cstep = t.cstep; a.lstep = t.lstep; a.Rr = t.Rr; a.Wl = t.Wl; a.row_img = (g.OH - 1) * t.lstep + t.Rr;
    a.g8 = t.g8; a.nblk = t.nblk; a.c_virtual = t.c_virtual;
    a.plane = t.plane;
    a.pitch = t.pitch; a.part = t.part; a.octet = t.octet;
    a.words_at = t.lds_bytes - 16;
    a.wr = t.wr;
    a.quads = (d.W + 3) / 4;
    a.wide = t.cstep == 1 && d.W >= 4 && t.Wl >= d.W + d.pad ? 1 : t.cstep == 1 && t.Wl == 1 && t.Rr == 1 && t.lstep == 1 && d.pad == 0 && a.OHW % 4 == 0 ? 2 : 0;
    const int bn = 16 * t.nt * (t.wr == 2 ? 2 : 4);
    a.n_ptiles = (int)((P + bn - 1) / bn);
    // (from the last position's first input row in the last channel to behind the last column that its cells take of the last row)
    auto passes_end = [&](int64_t p1) {
        const int64_t n = p1 / a.OHW, y = (p1 - n * a.OHW) / a.OW;
        return n * d.C * HW + (d.C - 1) * HW + (y + t.Rr) * t.cstep * d.W + (int64_t)t.Wl * t.cstep > (int64_t)N * d.C * HW;
    };
    int run_tiles = t.runs ? a.n_ptiles : 0;
    while (run_tiles > 0 && passes_end(std::min(run_tiles * (int64_t)bn, P) - 1)) --run_tiles;
    a.run_until = run_tiles * bn;
    a.n_mtiles = t.n_units / t.wr;
    a.n_units = t.n_units;
    a.groups = d.groups;
    a.wexp = t.wexp;
    a.small_sum = t.small_sum;
    a.stream_bytes = t.stream_bytes;
    a.in_ch4 = (int)(HW * 4); a.in_img = d.C * HW; a.in_group = g.Cg * HW; a.in_floats = (int64_t)N * d.C * HW;
    a.out_img = (int64_t)d.K * a.OHW; a.out_row = a.OHW;
    // what the kernel assumes
    if (t.plane > 1024 || t.plane % 64 || t.g8 < 1 || (int64_t)t.g8 * t.octet * 16 + 8 * t.plane > a.words_at || t.lds_bytes % 16 ||
        a.words_at < 4 * SCONV_MC_STORE_BYTES(t.mt, t.nt) || t.lds_bytes > 160 * 1024 || (int64_t)t.g8 * t.octet > 0xffff || t.n_units % t.wr ||
        (t.wr != 1 && t.wr != 2) || t.nt > t.nt_max || (a.wide == 1 && t.plane / t.Wl * a.quads > t.plane))
        return SCONV_ERR_PLAN;
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
    a.d_quads = make_fastdiv(a.quads, 4096);
    hipStream_t s = static_cast<hipStream_t>(stream);
#define X(M, NN) if (t.mt == M && t.nt == NN) return launch_mc_inst<M, NN>(a, (int)grid, t.lds_bytes, s, hip_err);
    X(2, 2) X(3, 2) X(4, 2) X(2, 4) X(3, 4) X(4, 4)
#undef X
    return SCONV_ERR_PLAN;
}

} // namespace sconv
