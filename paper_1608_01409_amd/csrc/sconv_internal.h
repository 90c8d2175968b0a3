// Internal declarations shared by the host code and the kernel launchers of libsconv.
#pragma once

#include <cstdint>
#include <vector>

#include "sconv.h"

namespace sconv {

// Nonzeros per straight-line group of the LDS kernel; (row, block) segments are padded to a multiple.
#define SCONV_PAIR_GROUP 4

struct Geometry {
    int Cg, Kg, Hp, Wp, OH, OW;
};

inline Geometry geometry(const sconv_desc &d)
{
    Geometry g;
    g.Cg = d.C / d.groups;
    g.Kg = d.K / d.groups;
    g.Hp = d.H + 2 * d.pad;
    g.Wp = d.W + 2 * d.pad;
    g.OH = (g.Hp - d.R) / d.stride + 1;
    g.OW = (g.Wp - d.S) / d.stride + 1;
    return g;
}

// Tiling of the LDS kernel, derived from a sconv_plan and the layer.
//
// LDS holds one block of `cb` input channels of `nt` images as
// [channel][cell][image]: `cell` runs over a Hl x Wl plane of the zero-padded
// image, `image` is innermost so that a lane reading `vec` consecutive floats
// reads `vec` images at one cell, always at an aligned address.  The row pitch
// is Wl = max(W + pad, OW): a read that falls into the right padding of a row
// lands on the left padding of the next one, which is zero as well.
// A workgroup computes a band of `band` output rows starting at row y0 and
// stages rows y0 .. y0 + band + R - 2 of the padded image; y below is relative
// to y0, so the packed offsets are the same for every band.
// A nonzero (c,r,s) of a row then reads, for flat output index
// F = pos*nt + image with pos = y*Wl + x, the float at
//   ((c_local*plane_cells + r*Wl + s)*nt) + F,
// i.e. the packed byte offset plus a per-lane constant.
struct LdsTiling {
    sconv_plan p;
    int vec;            // floats per lane per chunk: 4 if nt % 4 == 0 else 1
    int Wl, Hl;         // plane pitch and rows (Hl = band + R - 1 rows of the padded image)
    int n_bands;        // ceil(OH / band): bands of output rows, one workgroup each
    int plane_cells;    // Hl * Wl
    int pos_span;       // (band-1)*Wl + OW: positions a tile computes
    int pos_per_chunk;  // 64*vec / nt
    int n_chunks;       // ceil(pos_span / pos_per_chunk), <= cg*t
    int nblk;           // ceil(Cg / cb)
    int rg;             // row groups = waves / cg
    int nkt;            // K tiles per group
    int wave_slots;     // groups * nkt * rg
    int n_slabs;        // 64-float slabs per channel plane (staging granule)
    int n_bufs;         // LDS block buffers: 2 (double-buffered; 3 for the flow variant) unless the layer has fewer blocks
    int ctr_bytes_at;   // flow variant: byte offset in LDS of its per-block counters (nblk dwords), else 0
    int phase_cg;       // > 0: stride-1 form of a strided, unpadded layer whose blocks hold whole phases' channels
                        // (that many real channels per phase): staged straight from the caller's input
    int buf_stride_floats; // floats from one buffer to the next: block + zero page, multiple of 4
    int lds_bytes;      // dynamic LDS per workgroup
    unsigned zero_page; // byte offset, relative to a buffer, of its all-zero page (padding entries)
    int page_cells;     // size of that page in cells of nt floats
    int strip_rows;     // strip layout: rows of the block of positions one chunk covers (64 / strip), else 0
    int out_pos;        // floats from one output position to the next in the caller's layout (1 for NCHW)
    double us;          // what the cost model expects a launch to take (flat-stream tilings the search chose, else 0)
};

struct PackedLds {
    LdsTiling t;
    std::vector<uint64_t> pairs;   // low 32 bits: fp32 value bits; high 32: LDS byte offset
    std::vector<int32_t> seg_ptr;  // [wave_slot][nblk][rows_w + 1] -> index into pairs
    std::vector<int32_t> row_of;   // [wave_slot][rows_w] -> output channel or -1
};

// plan.kernel values that run the flat-stream kernel: 3 = a barrier per channel block, two block buffers;
// 4 = the flow variant, lds2_flow_bufs() buffers and per-block counters instead of barriers.  Same packing for both.
inline bool is_flat_kernel(int kernel) { return kernel == 3 || kernel == 4; }

// Packing for the flat-stream kernel (tiles of 4 images).  One stream per (wave slot, channel block)
// holding the nonzeros of all rows of the slot in that block, padded to whole chunks of 8 entries:
//   low 32 bits  fp32 value bits
//   high 32 bits (LDS byte offset / 16) << 16 | (row index inside the slot * t * 4)
// Padding entries have value +0.0 and point at the zero page.
#define SCONV_FLAT_CHUNK 8
// The kernel warms L2 with this many bytes of the stream beyond the point its scalar loads have reached (which is
// up to two chunks past a segment's end): the stream array carries that much padding behind its last segment.
#define SCONV_FLAT_WARM_BYTES 4096
struct PackedFlat {
    LdsTiling t;
    std::vector<uint64_t> pairs;
    std::vector<uint32_t> seg;       // [wave_slot][nblk] x (byte offset into pairs, number of chunks)
    std::vector<int32_t> row_of;     // [wave_slot][rows_w] -> output channel or -1
    std::vector<int32_t> store_tbl;  // [cg*t*64] -> (by*OW + ox)*4 inside a band, or -1
};

struct PackedDirect {
    std::vector<int32_t> rowptr;   // K+1
    std::vector<uint32_t> trip;    // 3 words per nonzero: value bits, goff, (dr<<16)|(ds&0xffff)
};

struct Canonical {
    std::vector<int32_t> rowptr, colidx, off;
    std::vector<float> val;
};

// Packing for the gather kernels (small launches), the same for every batch size.  Convolutions: rows padded to whole
// chunks, entry = (value bits, byte offset of (c, r, s) in the unpadded image << 3 | (31 - tap)); padding entries are
// (0, 0).  Layers the four-position kernel takes (gather4_fits): the entries between the first and the last channel of the
// tensor in whole chunks, low bits = tap, then the others one by one; per row (first entry, chunks, other entries).
// Fully connected layers (taps = 0): entry = (value bits, feature), rows not padded.
#define SCONV_GATHER_CHUNK 8
#define SCONV_GATHER_MAX_TAPS 31
#define SCONV_FC_GATHER_MAX_N 16384  // images: the grid's second dimension counts pieces of them
struct PackedGather {
    std::vector<uint64_t> ent;
    std::vector<int32_t> rowptr;   // [K + 1], in entries (gather4_fits: [K][3])
};
// What one wave of a gather kernel covers: t x 64 output positions (fully connected: t pieces of 4 images); split waves
// share a row.
struct GatherShape {
    int t, split;
    double us;                     // what the launch is expected to take
    double margin;                 // its time counts with this factor when kernels are compared: how far the model is trusted here
    double flat_us;                // its time with the factor that counts against the flat streams on the vector units alone (0: as above)
};
int pack_gather(const sconv_desc &d, const Canonical &c, PackedGather &out);
int pack_fc_gather(const sconv_desc &d, const Canonical &c, PackedGather &out);
bool gather_fits(const sconv_desc &d, int N);
bool gather4_fits(const sconv_desc &d);
bool gather4_flat(const sconv_desc &d, int N, int split);
bool fc_gather_fits(const sconv_desc &d, int N);
GatherShape choose_gather(const sconv_desc &d, int N, double avg_row_nnz, int max_row_nnz);
GatherShape choose_fc_gather(const sconv_desc &d, int N, double avg_row_nnz, int max_row_nnz);

// Tiling of the matrix-core kernel (rather dense layers).  The packing depends only on the layer: mt and nt may change
// from call to call.
struct MfmaTiling {
    bool phased;             // channels are phase images picked out of the input (unpadded strided layers)
    bool one_tap;            // one tap, stride 1: sconv_mfma_column_kernel can take it
    bool column = false;     // and takes it
    int mt = 0, nt = 0;      // a workgroup takes 32 * mt filters and 128 * nt positions
    int nt_max;              // 1 where 256 positions are too many for LDS, or 128 serve better
    int splits;              // workgroups along the channel blocks (partial sums, added by a launch of their own)
    int g8, nblk;            // channel octets staged per block, blocks
    int steps, steps_last, total_steps; // MFMA depth steps (two octets of one or two taps) of a block, the last block, all
    int c_virtual;           // channels of a group the kernel sees
    int cstep, lstep;        // input elements per cell, cells per output position
    int Rr, Sr, Wl;          // filter in cells, cells per staged row
    int plane;               // cells of an octet's plane in LDS (a multiple of 64)
    int n_tiles32;           // 32-row tiles per group, an even number
    int n_mtiles;            // workgroups along a group's filters
    int lds_bytes;
    double us;
};
// Offset of a channel that does not exist: bit 31 puts the lane offset out of range; the scalar offset, which the range check
// takes off the buffer's length, is 0.
#define SCONV_MFMA_NO_CHANNEL INT32_MIN
// Activations are staged times this and weights packed divided by it; a stored zero is packed as -0.
#define SCONV_MFMA_SCALE 65536.0f
// Rows of fewer nonzeros are summed over them (see the kernel); a layer may have one in SCONV_MFMA_SHORT_SHARE of them: each
// costs a workgroup a pass over its positions (2-3 us).
#define SCONV_MFMA_SHORT_ROW 4
#define SCONV_MFMA_SHORT_SHARE 16
// Up to so many nonzeros a row a sum on the matrix cores is no further from the exact one than the gather kernel's of four positions
// (relative 2-norm in 1e-8 on rectified normals: 48 3.8 / 4.8, 64 4.2 / 5.0, 80 4.6-4.9 / 4.8, 128 5.4 / 4.9; plain normals: 64 5.4 / 5.9, 80 5.9 / 5.9;
// at 72 one random layer with a bias had 4.1 / 3.9).
#define SCONV_MFMA_GATHER_ROW 48
// A sum in one chain on the matrix cores is no further from the exact one than the flat streams' in up to so many parts, and in up to twice as
// many where rows have at most SCONV_MFMA_CHAIN_ROW nonzeros: adding the parts up rounds as well (in 1e-8 on rectified normals, here / there: 64
// nonzeros 4.1 / 10.4 in one part, 6.9 in four and five, 7.5 in eleven; 256 7.1 / 9.8 in eight, 9.3 in eleven; fully connected 265 7.2 / 9.4 in
// twelve, 385 8.7 / 10.3 in sixteen; 512 in three parts 7.0 / 10.9 in fifteen).
#define SCONV_MFMA_CHAIN_ROW 512
#define SCONV_MFMA_CHAIN_PARTS 8
struct PackedMfma {
    std::vector<uint16_t> wfrag;  // [group][32-row tile][step][part][lane][8], one spare step behind
    std::vector<int32_t> uoff;    // [2 * steps] + [2 * steps_last]
    std::vector<int32_t> choff;   // phased only: per channel of whole octets
};
bool mfma_fits(const sconv_desc &d, int N, bool feature_major);
bool mfma_weight_ok(float v);
sconv_desc mfma_desc(const sconv_desc &d);
// The layer's tiling (mt, nt and us for a batch of N); false if the kernel cannot take the layer.
bool choose_mfma(const sconv_desc &d, int N, MfmaTiling &t);
// The same layer on the column kernel (t.one_tap), in at least so many parts; false, and not to be launched, if it cannot be cut so.
// The blocks depend only on the layer.
bool choose_mfma_column(const sconv_desc &d, int N, int min_splits, MfmaTiling &t);
int pack_mfma(const sconv_desc &d, const Canonical &c, const MfmaTiling &t, PackedMfma &out);

// Flat streams on the matrix cores (sconv_flat_mc.hip).  The packing depends only on the layer: nt and splits may change from
// call to call.
struct FlatMcTiling {
    bool phased;             // as in MfmaTiling
    bool runs;               // phased, stride a multiple of four: channel [input channel][row][column] of the phases, so that four
                             // channels of a cell lie side by side in the input; else [row][column][input channel]
    int mt = 0, nt = 0;      // a wave takes 16 * mt filters and 16 * nt positions
    int wr;                  // waves along the filters: 2 (then 2 along the positions) or 1 (then 4)
    int nt_max;              // 2 where 64 positions a wave are too many for LDS
    int splits;              // workgroups along the channel blocks (partial sums, added by a launch of their own)
    int g8, nblk;            // channel octets staged per block, blocks
    int c_virtual;           // channels of a group the kernel sees
    int cstep, lstep;        // input elements per cell, cells per output position
    int Rr, Sr, Wl;          // filter in cells, cells per staged row
    int plane;               // cells that are staged at most, a multiple of 64
    int pitch, part, octet;  // 16-byte units of LDS from one row of cells, high to low part, one channel octet to the next
    int n_units;             // waves' worth of filters per group, a multiple of wr
    int lds_bytes;
    int wexp;                // weights are packed times 2^wexp
    float small_sum;         // packed: sums below it are taken again where there are activations that have lost bits
    int64_t stream_bytes;
    double us;
};
// A record of a wave's stream: one matrix step.  [tile][high, low part][lane] 8 fp16 weights (the two a row keeps of each four
// channels of two octets), then per lane the weights' places (2 bits each, 16 bits a tile, 32 a pair of tiles) and the LDS
// address / 16 of the two octets it reads, 16 bits each (lane i of four those of tile i in steps that every tile has its own of).
#define SCONV_MC_RECORD(MT) ((MT) * 2048 + 64 * (((MT) + 1) / 2 * 4 + 4))
// What a wave's results take in LDS on their way out.
#define SCONV_MC_STORE_BYTES(MT, NT) (16 * (MT) * (16 * (NT) + 4) * 4)
// Where a wave has registers for totals, to which its accumulators are added every few steps.
#define SCONV_MC_TOTALS(MT, NT) ((MT) * (NT) <= 12)
struct PackedFlatMc {
    std::vector<uint8_t> stream;
    std::vector<int32_t> seg;     // [group][unit][block]: first record, shared steps | private steps << 16
    std::vector<int32_t> row_of;  // [group][unit][16 * mt]
    std::vector<int32_t> choff;   // phased only: per channel of whole octets
};
// A step that every tile has its own octets of against one that all share: four times the LDS reads.
#define SCONV_MC_PRIVATE_COST 1.5
// Nonzeros that the shortest row has, empty ones apart, for sums that are no further from 64 bits than those of the kernel they
// replace.  Relative error of a row in 1e-8, here / there, rectified normal inputs, the mean of 100 and more rows a length:
//   sums without totals (64 x 64 a wave) against the vector units' chains: 120 nonzeros 14.3 / 13.7, 150 15.4 / 15.3, 160 15.6 / 15.8
#define SCONV_MC_ROW 160
//   with totals against the chains: 50 9.3 / 9.0, 60 9.4 / 9.9, 70 9.7 / 10.8
#define SCONV_MC_FLUSHED_ROW 72
//   totals in up to three parts against chains in two parts: 120 10.4 / 10.3, 150 10.6 / 11.4; in four: 180 10.5 / 10.3,
//   210 10.5 / 10.8; so many per part of a flat-stream tiling that splits the channels
#define SCONV_MC_ROW_SPLIT 80
//   totals against the three-part kernel: 650 11.7 / 11.4, 700 11.8 / 12.0, 750 11.9 / 12.4
#define SCONV_MC_LONG_ROW 740
//   ... where that kernel splits the channels, per part: in two 1000 11.4 / 10.9, 1200 11.6 / 11.8; three 1800 12.0 / 11.8, 2000
//   12.4 / 12.6; four 2600 12.5 / 12.3, 2800 12.6 / 12.8
#define SCONV_MC_LONG_ROW_SPLIT 1100
// From this density on most octets are needed twice.
#define SCONV_MC_DENSE 0.35
bool flat_mc_weights_ok(const sconv_desc &d, const Canonical &c);
// The shortest row that is not empty; 0 if all are.
int shortest_row(const Canonical &c);
// Tiling and time of the layer on the matrix cores; flushed: with totals, whatever the rows' length.  False if it cannot take it.
bool choose_flat_mc(const sconv_desc &d, const Canonical &c, int N, bool flushed, FlatMcTiling &t);
int pack_flat_mc(const sconv_desc &d, const Canonical &c, FlatMcTiling &t, PackedFlatMc &out);

int validate_desc(const sconv_desc &d);
// rowptr starts at 0 and never falls, columns inside [0, Cg*R*S) and strictly ascending in each row
int validate_csr(const sconv_desc &d, const int32_t *rowptr, const int32_t *colidx);
// colidx -> off for a padded image stored in `layout` (a sconv_layout); the arrays are assumed valid
void lower_offsets(const sconv_desc &d, int layout, const int32_t *rowptr, const int32_t *colidx, int32_t *off);
int build_canonical_from_dense(const sconv_desc &d, const float *w, Canonical &out);
int build_canonical_from_arrays(const sconv_desc &d, const int32_t *rowptr, const int32_t *colidx,
                                const float *values, Canonical &out);

// Fill in a tiling for the LDS kernel (fields of `req` that are 0 are chosen).  N_hint is the
// batch size the choice is tuned for.  Returns SCONV_ERR_PLAN if the layer cannot use it.
// phase_cg > 0: d is the stride-1 form of a strided layer without padding, with that many real channels per
// phase; tilings whose blocks hold whole phases' channels can then be staged without the phase-image pass.
// wide: the input will be staged a cell per lane and the output stored four images at a time (feature-major
// activations); the cost model prices the landing of a block and the stores accordingly.
int make_lds_tiling(const sconv_desc &d, const sconv_plan &req, int N_hint, double avg_row_nnz, LdsTiling &out, int phase_cg = 0,
                    bool wide = false);
// The max_out distinct tilings the cost model ranks best, best first (out[0] is make_lds_tiling's choice).
int rank_lds_tilings(const sconv_desc &d, const sconv_plan &req, int N_hint, double avg_row_nnz, int max_out,
                     std::vector<LdsTiling> &out, int phase_cg = 0, bool wide = false);
// p.kernel selects the shape list: 1 = per-row streams, 3 = flat streams (nt must be 4)
bool lds_kernel_available(int vec, int t, int rows_w);

int pack_lds(const sconv_desc &d, const Canonical &c, const LdsTiling &t, PackedLds &out);
int unpack_lds(const sconv_desc &d, const PackedLds &p, Canonical &out);
int pack_flat(const sconv_desc &d, const Canonical &c, const LdsTiling &t, PackedFlat &out);
int unpack_flat(const sconv_desc &d, const PackedFlat &p, Canonical &out);
bool lds2_kernel_available(int t, int rows_w, int step); // step: 64 (flat lanes) or the strip width
int lds2_depth(int t, int rows_w);
int lds2_flow_bufs(); // block buffers the flow variant of the flat-stream kernel rotates through // read-ahead depth of a flat-stream shape, 0 if there is none
int pack_direct(const sconv_desc &d, const Canonical &c, PackedDirect &out);
int unpack_direct(const sconv_desc &d, const PackedDirect &p, Canonical &out);

// Strided layers on the LDS kernels.  With stride s the input rows that one filter row r touches are
// y*s + r: split r = r'*s + py and they become rows y + r' of the "phase image" py (every s-th row of the
// padded image, starting at py), and the same along x.  A strided layer is therefore a stride-1, pad-0 layer
// over Cg*s*s virtual channels (py, px, c: phase by phase) of size Hq x Wq = (OH + R' - 1) x (OW + S' - 1) with an R' x S'
// filter, R' = ceil(R/s): no input element is duplicated, only re-ordered (Section 2.1 allows any layout
// function f that is additive in the output position).  phase_desc gives that layer, phase_canonical its
// CSR; unphase_canonical maps offsets of the virtual layer back to the real one.
void phase_desc(const sconv_desc &d, sconv_desc &v);
int phase_canonical(const sconv_desc &d, const Canonical &c, Canonical &vc);
int unphase_canonical(const sconv_desc &d, const Canonical &vc, Canonical &out);

// Division of a small non-negative number by a divisor fixed per launch: a multiply-high with
// magic = ceil(2^32 / d), exact while n * d < 2^32 (the launcher checks the largest n of each use and passes
// magic = 0, meaning "divide", where that does not hold or d is 1).  The generic 32-bit division costs some 30
// instructions per use, and the kernel's first microsecond was mostly these.
struct FastDiv {
    unsigned d, magic;
};
inline FastDiv make_fastdiv(int d, int64_t n_max)
{
    FastDiv f;
    f.d = (unsigned)d;
    f.magic = (d > 1 && n_max * (int64_t)d < ((int64_t)1 << 32)) ? (unsigned)((((uint64_t)1 << 32) + d - 1) / (uint64_t)d) : 0u;
    return f;
}

// Device side (sconv_kernels.hip, sconv_gather.hip)
struct DeviceLds {
    void *pairs = nullptr, *seg_ptr = nullptr, *row_of = nullptr, *store_tbl = nullptr;
};
struct DeviceDirect {
    void *rowptr = nullptr, *trip = nullptr;
};
struct DeviceGather {
    void *ent = nullptr, *rowptr = nullptr;
    bool uploaded = false;
};
int launch_lds(const sconv_desc &d, const LdsTiling &t, const DeviceLds &dev, const float *in, float *out,
               int N, void *stream, int *hip_err);
// Bias and ReLU applied to the outputs (bias null = none).
struct Epilogue {
    const float *bias = nullptr;
    bool relu = false;
};
struct DeviceMfma {
    void *wfrag = nullptr, *uoff = nullptr, *choff = nullptr;
    bool uploaded = false;
    bool short_rows = false;      // there are rows of 1 to SCONV_MFMA_SHORT_ROW - 1 nonzeros
};
// feature_major: in_t[C][N] -> out_t[K][N] of a fully connected layer.  With t.splits > 1 `out` is a workspace of that many
// outputs, split_stride floats apart; launch_reduce adds them up afterwards.
int launch_mfma(const sconv_desc &d, const MfmaTiling &t, const DeviceMfma &dev, const DeviceDirect &direct, const float *in, float *out,
                int N, bool feature_major, const Epilogue &ep, int64_t split_stride, void *stream, int *hip_err);
int allow_full_lds(const void *kern, int *hip_err);
int launch_gather(const sconv_desc &d, const DeviceGather &dev, const GatherShape &gs, const float *in, float *out, int N,
                  const Epilogue &ep, void *stream, int *hip_err);
int launch_fc_gather(const sconv_desc &d, const DeviceGather &dev, const GatherShape &gs, const float *in_t, float *out_t, int N,
                     const Epilogue &ep, void *stream, int *hip_err);
// Where the flat-stream kernel finds its operands, in floats.  Input element (image i of tile m, channel c,
// position p = Y*W + X of the unpadded image): m*in_tile + i*in_img + c*in_ch + p*in_pos.  Output (image i
// of tile m, row k, band b, position q inside the band): m*out_tile + b*out_band + k*out_row + i*out_img +
// q*out_pos.  nchw_layout() gives the convolution's [N][C][H][W] -> [N][K][OH][OW].
struct Lds2Layout {
    // phase_stride > 1: the input is the strided layer's own [N][C][H][src_w] tensor and the kernel picks the
    // phase images out of it while staging (cell (Y, X) of phase (py, px) is input (Y*s + py, X*s + px));
    // the tiling's phase_cg real channels make up one phase of a group
    int phase_stride = 1, src_w = 0;
    int64_t in_tile, in_img, in_ch, in_pos;
    int64_t in_rec_fixed, in_rec_img, in_rec_tile; // bytes tile m with n valid images may read: fixed + n * img - m * tile
    int64_t out_tile, out_band, out_row, out_img, out_pos;
};
Lds2Layout nchw_layout(const sconv_desc &d, const LdsTiling &t);
int launch_flat_mc(const sconv_desc &d, const FlatMcTiling &t, const DeviceLds &dev, const float *in, float *out, int N, const Epilogue &ep,
                   int64_t split_stride, void *stream, int *hip_err);
// With t.p.splits > 1 `out` is a workspace of splits * split_stride floats that receives each part's partial
// results in the output's layout, and launch_reduce adds them up (and applies the epilogue) afterwards.
int launch_lds2(const sconv_desc &d, const LdsTiling &t, const DeviceLds &dev, const Lds2Layout &lay, const float *in,
                float *out, int N, const Epilogue &ep, int64_t split_stride, void *stream, int *hip_err);
int launch_reduce(const float *parts, float *out, int splits, int64_t rows, int64_t inner, int K, const Epilogue &ep,
                  void *stream, int *hip_err);
// out[n][k][..] = max(out + bias[k], 0) in place, for the paths that do not fuse it: rows of `inner` floats
int launch_epilogue(float *out, int64_t rows, int64_t inner, int K, const Epilogue &ep, void *stream, int *hip_err);

// in [N][C][H][W] -> q [N][C*s*s][Hq][Wq], zero padding written out
int launch_phase(const sconv_desc &d, const sconv_desc &v, const float *in, float *q, int N, void *stream, int *hip_err);
int launch_direct(const sconv_desc &d, const DeviceDirect &dev, const float *in, float *out, int N,
                  void *stream, int *hip_err);
// The library's static device scratch (SCONV_NOALLOC_SCRATCH_BYTES) on the current device: its address
// there, looked up once per device and remembered.
int static_scratch(void **base, size_t *bytes, int *hip_err);
int upload(const void *host, size_t bytes, void **dev, int *hip_err);
void release(void *dev);

// A pair of events that brackets work on one stream (for sconv_tune); stop waits for the stream.
struct StreamTimer {
    void *e0 = nullptr, *e1 = nullptr;
};
int timer_create(StreamTimer &t, int *hip_err);
int timer_start(StreamTimer &t, void *stream, int *hip_err);
int timer_stop_ms(StreamTimer &t, void *stream, float *ms, int *hip_err);
void timer_destroy(StreamTimer &t);

} // namespace sconv
