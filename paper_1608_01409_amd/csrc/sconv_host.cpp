// Host side of libsconv: descriptor and CSR validation, canonical offset lowering
// (Figure 2's colidx -> f(c,r,s)), choice of a tiling, and packing of the nonzeros
// into the order and units the kernels read.  No device work happens here.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <functional>
#include <numeric>
#include <thread>

#include "sconv_internal.h"

namespace sconv {

int validate_desc(const sconv_desc &d)
{
    if (d.C < 1 || d.H < 1 || d.W < 1 || d.K < 1 || d.R < 1 || d.S < 1) return SCONV_ERR_DESC;
    if (d.stride < 1 || d.pad < 0 || d.groups < 1) return SCONV_ERR_DESC;
    if (d.C % d.groups || d.K % d.groups) return SCONV_ERR_DESC;
    if ((int64_t)d.H + 2 * (int64_t)d.pad < d.R || (int64_t)d.W + 2 * (int64_t)d.pad < d.S) return SCONV_ERR_DESC;
    // offsets inside one (padded) image and one group's CSR columns must fit int32
    const int64_t Hp = (int64_t)d.H + 2 * d.pad, Wp = (int64_t)d.W + 2 * d.pad;
    if ((int64_t)d.C * Hp * Wp >= (int64_t)1 << 30) return SCONV_ERR_RANGE;
    if ((int64_t)(d.C / d.groups) * d.R * d.S >= (int64_t)1 << 30) return SCONV_ERR_RANGE;
    if ((int64_t)d.K * (d.C / d.groups) * d.R * d.S >= (int64_t)1 << 31) return SCONV_ERR_RANGE;
    if (d.R > 255 || d.S > 255 || d.pad > 255) return SCONV_ERR_RANGE;
    return SCONV_OK;
}

// Figure 2's layout function on the zero-padded image.  CHW: f(c,r,s) = (c*Hp + r)*Wp + s.  HWC (channel
// innermost): f(c,r,s) = (r*Wp + s)*C + c.  Both are additive in the position, which is all Section 2.1 asks.
void lower_offsets(const sconv_desc &d, int layout, const int32_t *rowptr, const int32_t *colidx, int32_t *off)
{
    const Geometry g = geometry(d);
    for (int k = 0; k < d.K; ++k) {
        const int grp = k / g.Kg;
        for (int j = rowptr[k]; j < rowptr[k + 1]; ++j) {
            const int col = colidx[j];
            const int s = col % d.S, r = (col / d.S) % d.R, ch = grp * g.Cg + col / (d.S * d.R);
            off[j] = layout == SCONV_LAYOUT_HWC ? (r * g.Wp + s) * d.C + ch : (ch * g.Hp + r) * g.Wp + s;
        }
    }
}

static void lower(const sconv_desc &d, Canonical &c)
{
    c.off.resize(c.colidx.size());
    lower_offsets(d, SCONV_LAYOUT_CHW, c.rowptr.data(), c.colidx.data(), c.off.data());
}

int validate_csr(const sconv_desc &d, const int32_t *rowptr, const int32_t *colidx)
{
    const Geometry g = geometry(d);
    const int64_t ncol = (int64_t)g.Cg * d.R * d.S;
    if (rowptr[0] != 0) return SCONV_ERR_CSR;
    for (int k = 0; k < d.K; ++k)
        if (rowptr[k + 1] < rowptr[k]) return SCONV_ERR_CSR;
    if (rowptr[d.K] > 0 && !colidx) return SCONV_ERR_NULL;
    for (int k = 0; k < d.K; ++k) {
        if ((int64_t)rowptr[k + 1] - rowptr[k] > ncol) return SCONV_ERR_CSR;
        for (int32_t j = rowptr[k]; j < rowptr[k + 1]; ++j) {
            if (colidx[j] < 0 || colidx[j] >= ncol) return SCONV_ERR_CSR;
            if (j > rowptr[k] && colidx[j] <= colidx[j - 1]) return SCONV_ERR_CSR;
        }
    }
    return SCONV_OK;
}

int build_canonical_from_dense(const sconv_desc &d, const float *w, Canonical &out)
{
    const Geometry g = geometry(d);
    const int64_t ncol = (int64_t)g.Cg * d.R * d.S;
    out.rowptr.assign(d.K + 1, 0);
    out.colidx.clear();
    out.val.clear();
    for (int k = 0; k < d.K; ++k) {
        const float *row = w + (int64_t)k * ncol;
        for (int64_t j = 0; j < ncol; ++j) {
            if (row[j] == 0.0f) continue; // +0 and -0 are pruned; NaN compares unequal and stays
            out.colidx.push_back((int32_t)j);
            out.val.push_back(row[j]);
        }
        out.rowptr[k + 1] = (int32_t)out.colidx.size();
    }
    lower(d, out);
    return SCONV_OK;
}

int build_canonical_from_arrays(const sconv_desc &d, const int32_t *rowptr, const int32_t *colidx,
                                const float *values, Canonical &out)
{
    const int rc = validate_csr(d, rowptr, colidx);
    if (rc) return rc;
    const int32_t nnz = rowptr[d.K];
    if (nnz > 0 && !values) return SCONV_ERR_NULL;
    out.rowptr.assign(rowptr, rowptr + d.K + 1);
    out.colidx.assign(colidx, colidx + nnz);
    out.val.assign(values, values + nnz);
    lower(d, out);
    return SCONV_OK;
}

// ------------------------------------------------------------------ tiling

static int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Row pitch of the LDS plane.  W + pad columns are enough for the reads: one that runs into the right
// padding of a row (X >= W + pad) lands on column X - pitch < pad of the next row, left padding, zero as
// well.  The pitch must also hold a whole output row, which is wider than that when pad > S - 1, and a
// whole filter row, so that two taps never share a cell (images narrower than the filter: both taps would
// read nothing but padding, yet the packing could no longer be decoded).
// With strips, lane l of a chunk sits on cell (l / strip) * pitch + l % strip; a pitch congruent to the strip
// width modulo 16 makes that congruent to l, so that the 64 lanes of a 16-byte read fall on the LDS banks
// exactly as 64 consecutive cells do (the natural pitch costs a third of the read rate in bank conflicts).
static int lds_pitch(const sconv_desc &d, int strip = 0)
{
    const Geometry g = geometry(d);
    int pitch = std::max(std::max(d.W + d.pad, g.OW), d.S);
    while (strip && (pitch - strip) % 16) ++pitch;
    return pitch;
}

static int fill_tiling(const sconv_desc &d, const sconv_plan &p, LdsTiling &t, int phase_cg = 0)
{
    const Geometry g = geometry(d);
    if (d.stride != 1) return SCONV_ERR_PLAN;
    if (p.nt < 1 || p.cb < 1 || p.waves < 1 || p.waves > 16 || p.cg < 1 || p.rows_w < 1 || p.t < 1) return SCONV_ERR_PLAN;
    if (p.band < 0 || p.band > g.OH) return SCONV_ERR_PLAN;
    if (p.waves % p.cg) return SCONV_ERR_PLAN;
    t.p = p;
    t.us = 0.0;
    if (!is_flat_kernel(p.kernel)) t.p.kernel = 1;
    const bool flat = is_flat_kernel(t.p.kernel), flow = t.p.kernel == 4;
    t.vec = (p.nt % 4 == 0) ? 4 : 1;
    if ((64 * t.vec) % p.nt) return SCONV_ERR_PLAN;
    if (p.strip < 0 || p.strip > 64 || (p.strip && !flat)) return SCONV_ERR_PLAN;
    if (flat) {
        if (p.nt != 4 || !lds2_kernel_available(p.t, p.rows_w, p.strip ? p.strip : 64)) return SCONV_ERR_PLAN;
    } else if (!lds_kernel_available(t.vec, p.t, p.rows_w)) {
        return SCONV_ERR_PLAN;
    }
    t.strip_rows = p.strip ? 64 / p.strip : 0;
    t.out_pos = 1;
    if (p.splits < 0 || (p.splits > 1 && !flat)) return SCONV_ERR_PLAN;
    if (t.p.splits == 0) t.p.splits = 1;
    if (t.p.band == 0) t.p.band = p.strip ? std::min(g.OH, p.cg * t.strip_rows) : g.OH;
    t.n_bands = ceil_div(g.OH, t.p.band);
    t.Wl = lds_pitch(d, p.strip);
    t.Hl = t.p.band + d.R - 1;
    t.plane_cells = t.Hl * t.Wl;
    t.pos_span = (t.p.band - 1) * t.Wl + g.OW;
    t.pos_per_chunk = 64 * t.vec / p.nt;
    t.n_chunks = ceil_div(t.pos_span, t.pos_per_chunk);
    if (p.strip) {
        // t strips of `strip` columns cover the width, cg blocks of strip_rows rows the band
        if (p.t * p.strip < g.OW || t.p.band > p.cg * t.strip_rows) return SCONV_ERR_PLAN;
        t.n_chunks = p.cg * p.t;
    } else if (t.n_chunks > p.cg * p.t) {
        return SCONV_ERR_PLAN;
    }
    if (p.cb > g.Cg) t.p.cb = g.Cg;
    t.nblk = ceil_div(g.Cg, t.p.cb);
    // A strided layer without padding can be staged straight from the caller's input when no channel block
    // straddles two phases (the virtual channels are ordered phase by phase, phase_cg real channels each)
    t.phase_cg = (phase_cg > 0 && flat && phase_cg % t.p.cb == 0) ? phase_cg : 0;
    if (t.p.splits > t.nblk) return SCONV_ERR_PLAN;
    // every part takes ceil(nblk / splits) blocks; fewer parts if the last ones would be empty
    t.p.splits = ceil_div(t.nblk, ceil_div(t.nblk, t.p.splits));
    t.rg = p.waves / p.cg;
    const int kt = t.rg * p.rows_w;
    t.nkt = ceil_div(g.Kg, kt);
    t.wave_slots = d.groups * t.nkt * t.rg;
    const int plane_floats = t.plane_cells * p.nt;
    t.n_slabs = ceil_div(plane_floats, 64);
    if (ceil_div(t.n_slabs, p.waves) > 4) return SCONV_ERR_PLAN; // slabs one wave stages per channel
    // LDS layout in floats: n_bufs x { [block: cb*plane_cells*nt] [zero page] }.  The zero
    // pages are cleared once per launch and never written.  A page serves three readers of the block in
    // front of it: the right padding of the very last row (pad*nt floats past the block), lanes past the
    // last valid position (their results are dropped), and the padding entries of the nonzero stream,
    // whose offset is the page's start, so that they multiply 0 by 0 for every lane and chunk: the page
    // has one cell more than the farthest cell a lane's chunk can start on (flat lanes: cg*t*64 cells;
    // strips: last row of the band, last column of the last strip).
    const int64_t block = (int64_t)t.p.cb * plane_floats;
    t.page_cells = p.strip ? (t.p.band - 1) * t.Wl + p.t * p.strip : p.cg * p.t * 64 * t.vec / p.nt;
    const int64_t page = (int64_t)t.page_cells * p.nt;
    if (page < (int64_t)d.pad * p.nt) return SCONV_ERR_PLAN;
    const int64_t stride = (block + page + 3) / 4 * 4;
    // barrier variant: two buffers; flow variant: its ring of buffers, and one counter per block behind them
    t.n_bufs = std::min(flow ? lds2_flow_bufs() : 2, t.nblk);
    const int64_t ctr_bytes = flow ? ((int64_t)t.nblk * 4 + 15) / 16 * 16 : 0;
    if (stride * t.n_bufs * 4 + ctr_bytes > 160 * 1024) return SCONV_ERR_PLAN;
    t.buf_stride_floats = (int)stride;
    t.ctr_bytes_at = flow ? (int)(stride * t.n_bufs * 4) : 0;
    t.lds_bytes = (int)(stride * t.n_bufs * 4 + ctr_bytes);
    t.zero_page = (unsigned)(block * 4);
    return SCONV_OK;
}

// Supported accumulator shapes; must match the instantiations in sconv_kernels.hip.
static const int kShapesV4[][2] = {{1, 8}, {2, 4}, {2, 8}, {3, 4}, {3, 6}, {3, 8}, {4, 4}, {4, 6}, {5, 4},
                                   {6, 2}, {6, 3}, {7, 2}, {7, 3}, {13, 1}, {14, 1}};
// read-ahead depth (stream entries in flight) of each shape above, as generated by gen_lds_loops.py
static const int kDepthV4[] = {4, 4, 2, 4, 2, 1, 2, 1, 1, 2, 1, 2, 1, 1, 1};

static int shape_depth(int vec, int t, int rows_w)
{
    if (vec != 4) return 1;
    for (size_t i = 0; i < sizeof(kDepthV4) / sizeof(kDepthV4[0]); ++i)
        if (kShapesV4[i][0] == t && kShapesV4[i][1] == rows_w) return kDepthV4[i];
    return 1;
}
static const int kShapesV1[][2] = {{1, 16}, {2, 16}, {3, 8}, {3, 16}, {4, 8}, {7, 8}, {13, 4}, {14, 4}};

bool lds_kernel_available(int vec, int t, int rows_w)
{
    if (vec == 4) {
        for (auto &s : kShapesV4)
            if (s[0] == t && s[1] == rows_w) return true;
    } else if (vec == 1) {
        for (auto &s : kShapesV1)
            if (s[0] == t && s[1] == rows_w) return true;
    }
    return false;
}

// Rough cost of a tiling in CU clocks; only used to rank candidates.
static double tiling_cost(const sconv_desc &d, const LdsTiling &t, int N, double avg_row_nnz)
{
    const Geometry g = geometry(d);
    const int n_tiles = ceil_div(N, t.p.nt);
    const double wgs = (double)n_tiles * d.groups * t.nkt * t.n_bands;
    const int by_lds = std::max(1, (160 * 1024) / (t.lds_bytes + 512));
    const int by_waves = std::max(1, 16 / t.p.waves);
    const int wpc = std::min(by_lds, by_waves);
    const double rows_per_wave = (double)g.Kg / (t.nkt * t.rg); // after dealing rows evenly
    // per-row streams: every (row, block) segment is padded to whole chunks of 4, 1.5 entries on average;
    // flat streams: every (wave, block) segment is padded to whole chunks of 8, 3.5 entries on average
    const bool flat = t.p.kernel == 3;
    const double seg_len = std::max(0.25, (flat ? rows_per_wave : 1.0) * avg_row_nnz / t.nblk);
    const double nnz_wave = rows_per_wave * avg_row_nnz * (seg_len + (flat ? 3.5 : 1.5)) / seg_len;
    const double fma_instr = t.p.t * t.vec;
    // SIMD-issue bound: waves on a SIMD run one after another; 4 clocks per wave instruction.
    // a shallow read-ahead ring leaves the wave waiting on LDS latency more often
    const double ring = 1.0 + 2.0 / (shape_depth(t.vec, t.p.t, t.p.rows_w) * t.p.t);
    const double simd = std::ceil(t.p.waves / 4.0) * nnz_wave * 4.0 * (fma_instr + 2.0) * ring;
    // LDS bound: clocks per wave read instruction.
    const double lds = t.p.waves * nnz_wave * t.p.t * (t.vec == 4 ? 4.3 : 2.4);
    // per segment fixed costs (pointer fetch, loop set-up, scalar latency), per wave, partly hidden
    const double seg = (double)t.nblk * (flat ? 4.0 : t.p.rows_w) * 60.0 * std::ceil(t.p.waves / 4.0);
    // loads stream in behind the multiply-adds; only the first block's load is exposed
    const double stage = (double)t.p.cb * t.plane_cells * t.p.nt * 4.0 / 32.0 + 3000.0 + t.nblk * 300.0;
    // fewer than four waves per SIMD hide each other's stalls less well
    const double occ = std::sqrt(16.0 / std::min(16, t.p.waves * wpc));
    const double wg = std::max(simd, lds) * occ + seg + stage;
    const double rounds = std::ceil(wgs / (256.0 * wpc));
    return rounds * wpc * wg;
}

// The same for the flat-stream kernel, in microseconds at 2.4 GHz; constants fitted to measured plan sweeps
// of the AlexNet layers at batch 256 (useful issue efficiency of the multiply-add loop, cost of a channel
// block's barrier and pipeline refill, cost of a workgroup's prologue and stores).
// wide: the layer's input is staged a cell per lane and its output stored four images at a time (feature-major
// activations): a block lands sooner and the stores of a workgroup take a fraction of the time.
static const double kWideFixed = 0.7;
static double tiling_cost_flat(const sconv_desc &d, const LdsTiling &t, int N, double avg_row_nnz, bool wide)
{
    const Geometry g = geometry(d);
    const int splits = std::max(1, t.p.splits);
    const int blocks = ceil_div(t.nblk, splits);              // channel blocks one workgroup walks
    const double wgs = (double)ceil_div(N, 4) * d.groups * t.nkt * t.n_bands * splits;
    const int by_lds = std::max(1, (160 * 1024) / (t.lds_bytes + 512));
    const int wpc = std::max(1, std::min(by_lds, 16 / t.p.waves));
    const double rows_wave = (double)g.Kg / (t.nkt * t.rg);
    const double entries = rows_wave * avg_row_nnz / splits + 1.5 * blocks; // segments are padded to fours
    const double cu_wgs = std::ceil(wgs / 256.0);             // workgroups one CU has to run ...
    const double m = std::min((double)wpc, cu_wgs);           // ... m of them side by side
    const double wps = t.p.waves * m / 4.0;                   // waves per SIMD
    double eff = wps >= 4 ? 0.78 : wps >= 3 ? 0.72 : wps >= 2 ? 0.68 : 0.42;
    // a shallow read-ahead ring (8 rows of 3 chunks leave registers for one entry ahead only) costs little: measured
    // on the 27x27 layer, 8 rows per wave beat 6 by 5 % in either variant, the longer streams outweighing it
    if (lds2_depth(t.p.t, t.p.rows_w) * t.p.t < 6) eff *= 0.99;
    const double simd_clk = t.p.waves * entries * (4.0 * t.p.t + 1.7); // VALU clocks per SIMD, one workgroup
    // per channel block: the barrier and the refill of the read pipeline, which a second workgroup on the CU
    // fills, and what the staging of the block (L2 to LDS, every workgroup its own copy) takes from the loop;
    // per workgroup: prologue and stores, partly filled by a second workgroup as well
    const double block_bytes = (double)t.p.cb * t.plane_cells * 16.0;
    // The flow variant pays no barrier: measured against the barrier variant on the same layers it gains about
    // 1000 clocks per block of the barrier variant (0.4-0.7 us per block on the 13x13 layers at any density)
    // and loses what its smaller blocks cost in padding.  Either variant issues the loads of the next block
    // when a block starts and cannot start that block before they have landed: a block lasts at least the
    // landing time, which binds at low density (measured: 3.3 us for 50 KB, 4.5 us for 74 KB per CU).
    const bool flow = t.p.kernel == 4;
    const double sync = flow ? 100.0 : 800.0 / m;
    // (a cell per lane: 0.7 us for the first bytes of a block, then 37 bytes per clock and CU)
    const double landing = wide ? 1700.0 + m * block_bytes / 37.0 : 4000.0 + m * block_bytes / 11.0;
    const double compute_block = m * simd_clk / eff / blocks;
    const double per_block = std::max(compute_block + sync + m * block_bytes / 120.0, landing);
    double group = blocks * per_block + (m >= 2 ? (t.p.waves >= 8 ? 8000.0 : 10500.0) : 14000.0) * (wide ? kWideFixed : 1.0);
    // Measured: the flow variant is the slower one (3-12 %) where a second workgroup on the CU already fills
    // the barrier's gaps and the blocks are only a few channels deep, where a block's arithmetic does not outlast its loads by a margin (its loads have
    // only the first chunks of a block to land in), and where there are too few blocks to rotate buffers.
    if (flow && ((m >= 2 && t.p.cb < 8) || blocks < 3 || compute_block < 1.5 * landing)) group *= 1.1;
    // (measured on the fully connected layers: with 16 waves 5-7 % behind the barrier variant and its larger blocks,
    // with 8 waves up to 10 % ahead)
    else if (flow && wide && t.p.waves >= 16) group *= 1.12;
    if (t.p.t >= 7) group /= 0.88;                            // shapes short of address registers
    double us = std::ceil(cu_wgs / m) * group / 2400.0;
    if (splits > 1) {
        // every part stores its partial results and a launch of its own adds them up
        const double out_bytes = 4.0 * N * d.K * g.OH * g.OW;
        us += 4.0 + splits * (out_bytes / (wide ? 6.0e6 : 3.5e6) + 0.3); // the reduction reads every part: bandwidth, and latency per part
    }
    return us;
}

static int search_lds_tilings(const sconv_desc &d, const sconv_plan &req, int N_hint, double avg_row_nnz, LdsTiling &out,
                              std::vector<std::pair<double, LdsTiling>> *all, int phase_cg = 0, bool wide = false);
// whether the library, left to itself, considers the flow variant of the flat-stream kernel
static const bool kFlowByDefault = true;

int make_lds_tiling(const sconv_desc &d, const sconv_plan &req, int N_hint, double avg_row_nnz, LdsTiling &out, int phase_cg, bool wide)
{
    return search_lds_tilings(d, req, N_hint, avg_row_nnz, out, nullptr, phase_cg, wide);
}

static bool same_tiling(const sconv_plan &a, const sconv_plan &b)
{
    return a.kernel == b.kernel && a.nt == b.nt && a.cb == b.cb && a.waves == b.waves && a.cg == b.cg &&
           a.rows_w == b.rows_w && a.t == b.t && a.band == b.band && a.strip == b.strip && a.splits == b.splits;
}

int rank_lds_tilings(const sconv_desc &d, const sconv_plan &req, int N_hint, double avg_row_nnz, int max_out,
                     std::vector<LdsTiling> &out, int phase_cg, bool wide)
{
    std::vector<std::pair<double, LdsTiling>> all;
    LdsTiling best;
    const int rc = search_lds_tilings(d, req, N_hint, avg_row_nnz, best, &all, phase_cg, wide);
    if (rc) return rc;
    std::stable_sort(all.begin(), all.end(), [](const std::pair<double, LdsTiling> &a, const std::pair<double, LdsTiling> &b) {
        return a.first < b.first;
    });
    out.clear();
    for (const auto &c : all) {
        if ((int)out.size() >= max_out) break;
        bool seen = false;
        for (const auto &o : out) seen = seen || same_tiling(o.p, c.second.p);
        if (!seen) out.push_back(c.second);
    }
    return out.empty() ? SCONV_ERR_PLAN : SCONV_OK;
}

static int search_lds_tilings(const sconv_desc &d, const sconv_plan &req, int N_hint, double avg_row_nnz, LdsTiling &out,
                              std::vector<std::pair<double, LdsTiling>> *all, int phase_cg, bool wide)
{
    const Geometry g = geometry(d);
    if (d.stride != 1) return SCONV_ERR_PLAN;
    const bool full = req.nt && req.cb && req.waves && req.cg && req.rows_w && req.t;
    if (full) {
        const int rc = fill_tiling(d, req, out, phase_cg);
        if (!rc && all) all->emplace_back(0.0, out);
        return rc;
    }
    if (req.strip && req.kernel && !is_flat_kernel(req.kernel)) return SCONV_ERR_PLAN;
    const int kinds[3] = {4, 3, 1};

    double best = -1;
    const int nts_big[] = {4, 8, 16}; // 8 and 16 only on request
    const int nts_small[] = {1, 2};
    const int *nts = N_hint >= 4 ? nts_big : nts_small;
    const int n_nts = N_hint >= 4 ? 3 : 2;
    // every (waves, rows_w, cb) for one choice of image tile, band, column group, chunk count and lane layout
    auto try_shapes = [&](int nt, int vec, int band, int cg, int T, int strip) {
        const int Wl = lds_pitch(d, strip);
        for (int waves : {4, 8, 16}) {
            if (req.waves && req.waves != waves) continue;
            if (waves % cg) continue;
            for (int ki = 0; ki < 3; ++ki)
            for (int rows_w = 1; rows_w <= 24; ++rows_w) {
                const int kind = kinds[ki];
                const bool flat = is_flat_kernel(kind);
                if (req.kernel && req.kernel != kind) continue;
                if (strip && !flat) continue;
                // left to itself the library uses flat streams for tiles of 4 images and per-row
                // streams only for the small-batch tiles the flat kernel does not cover
                if (!req.kernel && flat != (nt == 4)) continue;
                if (!req.kernel && kind == 4 && !kFlowByDefault) continue;
                if (flat ? (nt != 4 || !lds2_kernel_available(T, rows_w, strip ? strip : 64))
                         : !lds_kernel_available(vec, T, rows_w))
                    continue;
                if (req.rows_w && req.rows_w != rows_w) continue;
                for (int wpc_target : {1, 2, 4}) {
                    if (waves * wpc_target > 16) continue;
                    const int budget = 160 * 1024 / wpc_target - 256;
                    const int64_t per_ch = (int64_t)(band + d.R - 1) * Wl * nt * 4;
                    const int64_t page_cells = strip ? (band - 1) * Wl + T * strip : cg * T * 64 * vec / nt;
                    const int64_t fixed = page_cells * nt * 4 + 16;
                    int cb = g.Cg; // one block, one buffer, if it fits; else two buffers (flow: three)
                    if (fixed + per_ch * cb > budget) {
                        cb = (int)((budget / 2 - fixed) / per_ch);
                        // flow: as many buffers as the layer has blocks, up to its ring
                        for (int nb = 3; kind == 4 && nb <= lds2_flow_bufs() && (cb < 1 || ceil_div(g.Cg, cb) >= nb); ++nb)
                            cb = (int)(((budget - 128) / nb - fixed) / per_ch);
                    }
                    if (req.cb) cb = req.cb;
                    if (cb < 1) continue;
                    // even out the blocks
                    if (!req.cb) cb = ceil_div(g.Cg, ceil_div(g.Cg, cb));
                    // a strided layer staged straight from the input: blocks of whole phases' channels
                    if (!req.cb && phase_cg > 0 && flat) {
                        cb = std::min(cb, phase_cg);
                        while (phase_cg % cb) --cb;
                    }
                    // channel blocks of a tile shared by several workgroups, when there are too few tiles
                    static const int split_choices[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32};
                    for (int sp : split_choices) {
                        if (req.splits ? sp != 1 : (sp > 1 && !flat)) continue;
                        const int splits = req.splits ? req.splits : sp;
                        sconv_plan p = {kind, nt, cb, waves, cg, rows_w, T, band, strip, splits};
                        LdsTiling t;
                        if (fill_tiling(d, p, t, phase_cg) != SCONV_OK) continue;
                        if (!req.splits && t.p.splits != sp) continue; // the same as a smaller choice
                        const double c = flat ? tiling_cost_flat(d, t, N_hint, avg_row_nnz, wide)
                                                   : tiling_cost(d, t, N_hint, avg_row_nnz);
                        t.us = flat ? c : 0.0;
                        if (all) all->emplace_back(c, t);
                        if (best < 0 || c < best) {
                            best = c;
                            out = t;
                        }
                    }
                }
            }
        }
    };

    for (int a = 0; a < n_nts; ++a) {
        const int nt = nts[a];
        if (req.nt && req.nt != nt) continue;
        if (!req.nt && nt > 4) continue;
        if (nt > 1 && nt > N_hint) continue;
        const int vec = nt % 4 == 0 ? 4 : 1;
        int last_band = 0;
        for (int nb = 1; nb <= 8 && nb <= g.OH && !req.strip; ++nb) {
            const int band = req.band ? req.band : ceil_div(g.OH, nb);
            if (band == last_band) continue; // same band height as the previous count
            last_band = band;
            const int pos_span = (band - 1) * lds_pitch(d) + g.OW;
            const int n_chunks = ceil_div(pos_span, 64 * vec / nt);
            for (int cg = 1; cg <= 4; ++cg) {
                if (req.cg && req.cg != cg) continue;
                const int T = ceil_div(n_chunks, cg);
                if (req.t && req.t != T) continue;
                if (!req.cg && (cg - 1) * T >= n_chunks) continue; // a wave of the column group without positions
                try_shapes(nt, vec, band, cg, T, 0);
            }
            if (req.band) break;
        }
        // strips: t blocks of (64 / strip) rows x strip columns side by side, cg such rows of blocks
        if (nt != 4) continue;
        for (int strip : {7, 8, 9}) {
            if (req.strip && req.strip != strip) continue;
            const int T = ceil_div(g.OW, strip), bh = 64 / strip;
            if (req.t && req.t != T) continue;
            for (int cg = 1; cg <= 4; ++cg) {
                if (req.cg && req.cg != cg) continue;
                const int nb = ceil_div(g.OH, cg * bh);
                const int band = req.band ? req.band : ceil_div(g.OH, nb);
                if (band > cg * bh) continue;
                try_shapes(nt, vec, band, cg, T, strip);
            }
        }
    }
    return best < 0 ? SCONV_ERR_PLAN : SCONV_OK;
}

// ------------------------------------------------------------------ packing

// Rows of one group are dealt to the group's wave slots in descending order of their nonzero count,
// boustrophedon, so that every wave (which owns rows_w rows for the whole kernel) gets about the same
// number of nonzeros even when the row lengths are skewed; empty rows are dealt like any other row
// and simply produce empty segments.
int pack_lds(const sconv_desc &d, const Canonical &c, const LdsTiling &t, PackedLds &out)
{
    const Geometry g = geometry(d);
    const int rows_w = t.p.rows_w, cb = t.p.cb, nt = t.p.nt;
    const int waves_per_group = t.nkt * t.rg;
    out.t = t;
    out.row_of.assign((size_t)t.wave_slots * rows_w, -1);
    for (int grp = 0; grp < d.groups; ++grp) {
        std::vector<int> rows(g.Kg);
        std::iota(rows.begin(), rows.end(), grp * g.Kg);
        std::stable_sort(rows.begin(), rows.end(), [&](int a, int b) {
            return c.rowptr[a + 1] - c.rowptr[a] > c.rowptr[b + 1] - c.rowptr[b];
        });
        for (int i = 0; i < g.Kg; ++i) {
            const int round = i / waves_per_group, posn = i % waves_per_group;
            const int w = (round & 1) ? waves_per_group - 1 - posn : posn;
            if (round >= rows_w) return SCONV_ERR_PLAN; // cannot happen: nkt*rg*rows_w >= Kg
            out.row_of[((size_t)grp * waves_per_group + w) * rows_w + round] = rows[i];
        }
    }
    out.seg_ptr.assign((size_t)t.wave_slots * t.nblk * (rows_w + 1), 0);
    out.pairs.clear();
    out.pairs.reserve(c.val.size() + c.val.size() / 4);
    size_t real = 0;
    for (int ws = 0; ws < t.wave_slots; ++ws) {
        for (int b = 0; b < t.nblk; ++b) {
            int32_t *sp = &out.seg_ptr[((size_t)ws * t.nblk + b) * (rows_w + 1)];
            for (int i = 0; i < rows_w; ++i) {
                sp[i] = (int32_t)out.pairs.size();
                const int k = out.row_of[(size_t)ws * rows_w + i];
                if (k < 0) continue;
                const int grp = k / g.Kg;
                for (int j = c.rowptr[k]; j < c.rowptr[k + 1]; ++j) {
                    // canonical offset -> (absolute channel, r, s)
                    const int off = c.off[j];
                    const int s = off % g.Wp, r = (off / g.Wp) % g.Hp, ca = off / (g.Wp * g.Hp);
                    const int cl = ca - grp * g.Cg - b * cb;
                    if (cl < 0 || cl >= cb) continue;
                    const uint32_t byte_off = (uint32_t)(((int64_t)cl * t.plane_cells + r * t.Wl + s) * nt * 4);
                    uint32_t vb;
                    std::memcpy(&vb, &c.val[j], 4);
                    out.pairs.push_back((uint64_t)vb | ((uint64_t)byte_off << 32));
                    ++real;
                }
                // pad the segment to whole groups: value +0.0 at the all-zero page
                while ((out.pairs.size() - (size_t)sp[i]) % SCONV_PAIR_GROUP) out.pairs.push_back((uint64_t)t.zero_page << 32);
            }
            sp[rows_w] = (int32_t)out.pairs.size();
        }
    }
    if (real != c.val.size()) return SCONV_ERR_PLAN;
    // the kernel prefetches up to three chunks past the stream it is working on
    for (int i = 0; i < 3 * SCONV_PAIR_GROUP; ++i) out.pairs.push_back((uint64_t)t.zero_page << 32);
    return SCONV_OK;
}

// Rows of one group dealt to the group's wave slots for the flat-stream kernel.  Every wave of a workgroup
// meets the others at a barrier after each channel block, so what has to be even is the number of nonzeros a
// slot holds in EACH block, not only its total.  Greedy: rows in descending order of their nonzero count,
// each to the slot (with a free row) whose fullest block stays smallest, ties to the smaller total.  Rows
// without nonzeros are dealt like any other and fill what is left.
static int deal_rows(const sconv_desc &d, const Canonical &c, const LdsTiling &t, std::vector<int32_t> &row_of)
{
    const Geometry g = geometry(d);
    const int rows_w = t.p.rows_w, nblk = t.nblk, cb = t.p.cb;
    const int slots = t.nkt * t.rg;
    row_of.assign((size_t)t.wave_slots * rows_w, -1);
    std::vector<int> per_blk((size_t)g.Kg * nblk);
    std::vector<int64_t> load((size_t)slots * nblk), total(slots);
    std::vector<int> used(slots);
    for (int grp = 0; grp < d.groups; ++grp) {
        std::fill(per_blk.begin(), per_blk.end(), 0);
        for (int i = 0; i < g.Kg; ++i) {
            const int k = grp * g.Kg + i;
            for (int j = c.rowptr[k]; j < c.rowptr[k + 1]; ++j) {
                const int ca = c.off[j] / (g.Wp * g.Hp);
                per_blk[(size_t)i * nblk + (ca - grp * g.Cg) / cb]++;
            }
        }
        std::vector<int> rows(g.Kg);
        std::iota(rows.begin(), rows.end(), 0);
        std::stable_sort(rows.begin(), rows.end(), [&](int a, int b) {
            const int ka = grp * g.Kg + a, kb = grp * g.Kg + b;
            return c.rowptr[ka + 1] - c.rowptr[ka] > c.rowptr[kb + 1] - c.rowptr[kb];
        });
        std::fill(load.begin(), load.end(), 0);
        std::fill(total.begin(), total.end(), 0);
        std::fill(used.begin(), used.end(), 0);
        for (int i : rows) {
            const int *r = &per_blk[(size_t)i * nblk];
            int best = -1;
            int64_t best_max = 0, best_tot = 0;
            for (int s2 = 0; s2 < slots; ++s2) {
                if (used[s2] >= rows_w) continue;
                int64_t mx = 0;
                for (int b = 0; b < nblk; ++b) mx = std::max(mx, load[(size_t)s2 * nblk + b] + r[b]);
                if (best < 0 || mx < best_max || (mx == best_max && total[s2] < best_tot)) {
                    best = s2;
                    best_max = mx;
                    best_tot = total[s2];
                }
            }
            if (best < 0) return SCONV_ERR_PLAN; // cannot happen: slots * rows_w >= Kg
            for (int b = 0; b < nblk; ++b) {
                load[(size_t)best * nblk + b] += r[b];
                total[best] += r[b];
            }
            row_of[((size_t)grp * slots + best) * rows_w + used[best]++] = grp * g.Kg + i;
        }
    }
    return SCONV_OK;
}

int pack_flat(const sconv_desc &d, const Canonical &c, const LdsTiling &t, PackedFlat &out)
{
    const Geometry g = geometry(d);
    const int rows_w = t.p.rows_w, cb = t.p.cb;
    if (t.p.nt != 4 || rows_w * t.p.t * 4 > 256 || t.zero_page >= (1u << 20) || t.zero_page % 16) return SCONV_ERR_PLAN;
    out.t = t;
    int rc = deal_rows(d, c, t, out.row_of);
    if (rc) return rc;
    out.seg.assign((size_t)t.wave_slots * t.nblk * 2 + 2, 0); // one spare entry: the kernel looks one block ahead
    out.pairs.clear();
    out.pairs.reserve(c.val.size() + (size_t)t.wave_slots * t.nblk * 4);
    const uint64_t pad_entry = (uint64_t)((t.zero_page / 16) << 16) << 32;
    size_t real = 0;
    // nonzeros of a row by block: walk each row once per slot, bucketing by channel block
    std::vector<std::vector<uint64_t>> bucket(t.nblk);
    for (int ws = 0; ws < t.wave_slots; ++ws) {
        for (auto &b : bucket) b.clear();
        for (int i = 0; i < rows_w; ++i) {
            const int k = out.row_of[(size_t)ws * rows_w + i];
            if (k < 0) continue;
            const int grp = k / g.Kg;
            for (int j = c.rowptr[k]; j < c.rowptr[k + 1]; ++j) {
                const int off = c.off[j];
                const int s = off % g.Wp, r = (off / g.Wp) % g.Hp, ca = off / (g.Wp * g.Hp);
                const int cl_all = ca - grp * g.Cg;
                const int b = cl_all / cb, cl = cl_all - b * cb;
                const uint32_t byte_off = (uint32_t)(((int64_t)cl * t.plane_cells + r * t.Wl + s) * 16);
                if (byte_off >= t.zero_page) return SCONV_ERR_PLAN;
                uint32_t vb;
                std::memcpy(&vb, &c.val[j], 4);
                bucket[b].push_back((uint64_t)vb | ((uint64_t)(((byte_off / 16) << 16) | (uint32_t)(i * t.p.t * 4)) << 32));
                ++real;
            }
        }
        for (int b = 0; b < t.nblk; ++b) {
            // entries in ascending LDS offset: rows that share a column sit next to each other
            std::stable_sort(bucket[b].begin(), bucket[b].end(), [](uint64_t x, uint64_t y) { return (x >> 48) < (y >> 48); });
            // The segment in whole chunks of 8 entries.  Its length is first rounded up to a multiple of 4; an
            // odd number of fours puts the first four into a chunk of their own, whose other four entries the
            // kernel never executes (flag in bit 31 of the chunk count), so that at most 3 entries of a
            // segment are idle instead of 7.
            const size_t start = out.pairs.size();
            const size_t len = bucket[b].size(), fours = (len + 3) / 4;
            const bool half = fours % 2 == 1;
            size_t taken = 0;
            if (half) {
                for (; taken < 4 && taken < len; ++taken) out.pairs.push_back(bucket[b][taken]);
                while ((out.pairs.size() - start) % SCONV_FLAT_CHUNK) out.pairs.push_back(pad_entry);
            }
            out.pairs.insert(out.pairs.end(), bucket[b].begin() + (long)taken, bucket[b].end());
            while ((out.pairs.size() - start) % SCONV_FLAT_CHUNK) out.pairs.push_back(pad_entry);
            if (start * 8 >= ((uint64_t)1 << 32)) return SCONV_ERR_RANGE;
            const size_t chunks = (out.pairs.size() - start) / SCONV_FLAT_CHUNK;
            if (chunks >= ((size_t)1 << 24)) return SCONV_ERR_RANGE;
            out.seg[((size_t)ws * t.nblk + b) * 2] = (uint32_t)(start * 8);
            out.seg[((size_t)ws * t.nblk + b) * 2 + 1] = (uint32_t)chunks | (half ? 0x80000000u : 0u);
        }
    }
    if (real != c.val.size()) return SCONV_ERR_PLAN;
    // the kernel loads two chunks past the segment it is working on, and warms L2 with what follows those
    for (int i = 0; i < 3 * SCONV_FLAT_CHUNK + SCONV_FLAT_WARM_BYTES / 8; ++i) out.pairs.push_back(pad_entry);
    // store offsets of the positions a group of cg waves covers
    const int npos = t.p.cg * t.p.t * 64;
    out.store_tbl.assign(npos, -1);
    for (int pos = 0; pos < npos; ++pos) {
        int by = pos / t.Wl, ox = pos % t.Wl;
        if (t.p.strip) { // [wave of the column group][chunk = strip][lane = row * strip + column]
            const int cgi = pos / (t.p.t * 64), ch = pos / 64 % t.p.t, lane = pos % 64;
            const int br = lane / t.p.strip;
            by = br < t.strip_rows ? cgi * t.strip_rows + br : t.p.band;
            ox = ch * t.p.strip + lane % t.p.strip;
        }
        if (by < t.p.band && ox < g.OW) out.store_tbl[pos] = (by * g.OW + ox) * 4 * t.out_pos;
    }
    return SCONV_OK;
}

static void sort_rows_by_offset(const sconv_desc &d, std::vector<std::vector<std::pair<int32_t, float>>> &rows,
                                Canonical &out)
{
    out.rowptr.assign(d.K + 1, 0);
    out.off.clear();
    out.val.clear();
    out.colidx.clear();
    for (int k = 0; k < d.K; ++k) {
        auto &r = rows[k];
        std::stable_sort(r.begin(), r.end(), [](const std::pair<int32_t, float> &a, const std::pair<int32_t, float> &b) {
            return a.first < b.first;
        });
        for (auto &e : r) {
            out.off.push_back(e.first);
            out.val.push_back(e.second);
        }
        out.rowptr[k + 1] = (int32_t)out.off.size();
    }
}

int unpack_lds(const sconv_desc &d, const PackedLds &p, Canonical &out)
{
    const Geometry g = geometry(d);
    const LdsTiling &t = p.t;
    const int rows_w = t.p.rows_w;
    std::vector<std::vector<std::pair<int32_t, float>>> rows(d.K);
    for (int ws = 0; ws < t.wave_slots; ++ws) {
        for (int b = 0; b < t.nblk; ++b) {
            const int32_t *sp = &p.seg_ptr[((size_t)ws * t.nblk + b) * (rows_w + 1)];
            for (int i = 0; i < rows_w; ++i) {
                const int k = p.row_of[(size_t)ws * rows_w + i];
                if (k < 0) {
                    if (sp[i + 1] != sp[i]) return SCONV_ERR_CSR;
                    continue;
                }
                const int grp = k / g.Kg;
                for (int j = sp[i]; j < sp[i + 1]; ++j) {
                    const uint32_t vb = (uint32_t)(p.pairs[j] & 0xffffffffu);
                    const uint32_t byte_off = (uint32_t)(p.pairs[j] >> 32);
                    if (byte_off >= t.zero_page) continue; // group padding
                    const int cell = (int)(byte_off / (4u * t.p.nt));
                    const int cl = cell / t.plane_cells, rem = cell % t.plane_cells;
                    const int r = rem / t.Wl, s = rem % t.Wl;
                    const int ca = grp * g.Cg + b * t.p.cb + cl;
                    float v;
                    std::memcpy(&v, &vb, 4);
                    rows[k].push_back({((ca * g.Hp) + r) * g.Wp + s, v});
                }
            }
        }
    }
    sort_rows_by_offset(d, rows, out);
    return SCONV_OK;
}

int unpack_flat(const sconv_desc &d, const PackedFlat &p, Canonical &out)
{
    const Geometry g = geometry(d);
    const LdsTiling &t = p.t;
    const int rows_w = t.p.rows_w;
    std::vector<std::vector<std::pair<int32_t, float>>> rows(d.K);
    for (int ws = 0; ws < t.wave_slots; ++ws) {
        for (int b = 0; b < t.nblk; ++b) {
            const size_t start = p.seg[((size_t)ws * t.nblk + b) * 2] / 8;
            const size_t n = (size_t)(p.seg[((size_t)ws * t.nblk + b) * 2 + 1] & 0x7fffffffu) * SCONV_FLAT_CHUNK;
            for (size_t j = start; j < start + n; ++j) {
                const uint32_t vb = (uint32_t)(p.pairs[j] & 0xffffffffu);
                const uint32_t w1 = (uint32_t)(p.pairs[j] >> 32);
                const uint32_t byte_off = (w1 >> 16) * 16;
                if (byte_off >= t.zero_page) continue; // chunk padding
                const int i = (int)(w1 & 0xffffu) / (t.p.t * 4);
                if (i >= rows_w) return SCONV_ERR_CSR;
                const int k = p.row_of[(size_t)ws * rows_w + i];
                if (k < 0) return SCONV_ERR_CSR;
                const int grp = k / g.Kg;
                const int cell = (int)(byte_off / 16u);
                const int cl = cell / t.plane_cells, rem = cell % t.plane_cells;
                const int r = rem / t.Wl, sx = rem % t.Wl;
                const int ca = grp * g.Cg + b * t.p.cb + cl;
                float v;
                std::memcpy(&v, &vb, 4);
                rows[k].push_back({((ca * g.Hp) + r) * g.Wp + sx, v});
            }
        }
    }
    sort_rows_by_offset(d, rows, out);
    return SCONV_OK;
}

// ------------------------------------------------------------------ strided layers as phase images

void phase_desc(const sconv_desc &d, sconv_desc &v)
{
    const Geometry g = geometry(d);
    const int s = d.stride;
    v = d;
    v.C = d.C * s * s;
    v.R = ceil_div(d.R, s);
    v.S = ceil_div(d.S, s);
    v.H = g.OH + v.R - 1;
    v.W = g.OW + v.S - 1;
    v.stride = 1;
    v.pad = 0;
}

int phase_canonical(const sconv_desc &d, const Canonical &c, Canonical &vc)
{
    const Geometry g = geometry(d);
    sconv_desc v;
    phase_desc(d, v);
    const Geometry gv = geometry(v);
    const int s = d.stride;
    std::vector<std::vector<std::pair<int32_t, float>>> rows(d.K);
    for (int k = 0; k < d.K; ++k) {
        const int grp = k / g.Kg;
        for (int j = c.rowptr[k]; j < c.rowptr[k + 1]; ++j) {
            const int off = c.off[j];
            const int t = off % g.Wp, r = (off / g.Wp) % g.Hp, ca = off / (g.Wp * g.Hp);
            const int cl = ca - grp * g.Cg;
            const int va = grp * gv.Cg + ((r % s) * s + t % s) * g.Cg + cl; // phase by phase, the group's channels inside
            rows[k].push_back({(va * gv.Hp + r / s) * gv.Wp + t / s, c.val[j]});
        }
    }
    sort_rows_by_offset(v, rows, vc);
    // colidx of the virtual layer, for completeness: (v_local*R' + r')*S' + t'
    vc.colidx.resize(vc.off.size());
    for (int k = 0; k < d.K; ++k) {
        const int grp = k / g.Kg;
        for (int j = vc.rowptr[k]; j < vc.rowptr[k + 1]; ++j) {
            const int off = vc.off[j];
            const int t = off % gv.Wp, r = (off / gv.Wp) % gv.Hp, va = off / (gv.Wp * gv.Hp);
            vc.colidx[j] = ((va - grp * gv.Cg) * v.R + r) * v.S + t;
        }
    }
    return SCONV_OK;
}

int unphase_canonical(const sconv_desc &d, const Canonical &vc, Canonical &out)
{
    const Geometry g = geometry(d);
    sconv_desc v;
    phase_desc(d, v);
    const Geometry gv = geometry(v);
    const int s = d.stride;
    std::vector<std::vector<std::pair<int32_t, float>>> rows(d.K);
    for (int k = 0; k < d.K; ++k) {
        const int grp = k / g.Kg;
        for (int j = vc.rowptr[k]; j < vc.rowptr[k + 1]; ++j) {
            const int off = vc.off[j];
            const int t2 = off % gv.Wp, r2 = (off / gv.Wp) % gv.Hp, va = off / (gv.Wp * gv.Hp);
            const int vl = va - grp * gv.Cg;
            const int cl = vl % g.Cg, px = (vl / g.Cg) % s, py = vl / (g.Cg * s);
            const int r = r2 * s + py, t = t2 * s + px;
            if (r >= d.R || t >= d.S) return SCONV_ERR_CSR;
            rows[k].push_back({((grp * g.Cg + cl) * g.Hp + r) * g.Wp + t, vc.val[j]});
        }
    }
    sort_rows_by_offset(d, rows, out);
    return SCONV_OK;
}

// Direct kernel: per nonzero the value, the offset of (c, r-pad, s-pad) in the UNPADDED image
// (may be negative), and (r-pad, s-pad) for the bounds test that stands in for the zero padding.
int pack_direct(const sconv_desc &d, const Canonical &c, PackedDirect &out)
{
    const Geometry g = geometry(d);
    out.rowptr = c.rowptr;
    out.trip.resize(c.val.size() * 3);
    for (size_t j = 0; j < c.val.size(); ++j) {
        const int off = c.off[j];
        const int s = off % g.Wp, r = (off / g.Wp) % g.Hp, ca = off / (g.Wp * g.Hp);
        const int dr = r - d.pad, ds = s - d.pad;
        const int32_t goff = (ca * d.H + dr) * d.W + ds;
        uint32_t vb;
        std::memcpy(&vb, &c.val[j], 4);
        out.trip[3 * j + 0] = vb;
        out.trip[3 * j + 1] = (uint32_t)goff;
        out.trip[3 * j + 2] = ((uint32_t)(dr & 0xffff) << 16) | (uint32_t)(ds & 0xffff);
    }
    return SCONV_OK;
}

int unpack_direct(const sconv_desc &d, const PackedDirect &p, Canonical &out)
{
    const Geometry g = geometry(d);
    std::vector<std::vector<std::pair<int32_t, float>>> rows(d.K);
    for (int k = 0; k < d.K; ++k) {
        for (int j = p.rowptr[k]; j < p.rowptr[k + 1]; ++j) {
            const uint32_t vb = p.trip[3 * (size_t)j];
            const int32_t goff = (int32_t)p.trip[3 * (size_t)j + 1];
            const uint32_t rs = p.trip[3 * (size_t)j + 2];
            const int dr = (int16_t)(rs >> 16), ds = (int16_t)(rs & 0xffff);
            const int ca = (goff - dr * d.W - ds) / (d.H * d.W);
            float v;
            std::memcpy(&v, &vb, 4);
            rows[k].push_back({((ca * g.Hp) + dr + d.pad) * g.Wp + ds + d.pad, v});
        }
    }
    sort_rows_by_offset(d, rows, out);
    return SCONV_OK;
}

// ------------------------------------------------------------------ gather kernels (small launches)

// The four-position kernel: neighbours in a row are neighbours in memory, and the four words of a lane stay inside the
// tensor for every tap of every channel but the first and the last.
bool gather4_fits(const sconv_desc &d)
{
    return d.stride == 1 && d.C >= 3 && (int64_t)d.H * d.W > (int64_t)d.pad * d.W + d.pad + 2;
}

// Its fours of positions are counted through the image instead of through each row, where that leaves the fullest CU a workgroup
// less: 441 random calls 1.066x, 37 more than 2 % slower, 8 more than 5 %.  With fewer workgroups but no round of them less it was 0.988x over
// 1005 (422 more than 2 % slower, 57 more than 5 %; 43 more than 5 % faster).  (Fewer than four positions a row would pass more than one
// row's end.)
bool gather4_flat(const sconv_desc &d, int N, int split)
{
    const Geometry g = geometry(d);
    const int rows = split >= 4 ? 1 : 4 / split;
    auto rounds = [&](int64_t fours) { return ((N * fours + 63) / 64 * ceil_div(d.K, rows) + 255) / 256; };
    return g.OW == d.W && g.OW >= 4 && rounds(ceil_div(g.OH * g.OW, 4)) < rounds((int64_t)g.OH * ceil_div(g.OW, 4));
}

int pack_gather(const sconv_desc &d, const Canonical &c, PackedGather &out)
{
    const Geometry g = geometry(d);
    const bool four = gather4_fits(d);
    out.ent.clear();
    out.ent.reserve(c.val.size() + (size_t)d.K * SCONV_GATHER_CHUNK);
    out.rowptr.assign(four ? (size_t)3 * d.K : (size_t)d.K + 1, 0);
    // Filter rows and columns that some output position has inside the image.  The others (a filter larger than the image)
    // meet padding only: every position masks them, but r rows below the first may lie beyond the buffer, whose range check
    // takes the scalar offset off the record's length.  Their entries point at the channel's first element instead.
    auto seen = [&](int tap, int outputs, int size) {
        for (int y = 0; y < outputs; ++y)
            if (y * d.stride - d.pad + tap >= 0 && y * d.stride - d.pad + tap < size) return true;
        return false;
    };
    std::vector<char> row_seen(d.R), col_seen(d.S);
    for (int r = 0; r < d.R; ++r) row_seen[r] = seen(r, g.OH, d.H);
    for (int s = 0; s < d.S; ++s) col_seen[s] = seen(s, g.OW, d.W);
    // control word of every column of group 0; a group further on adds its channels' bytes
    std::vector<uint32_t> ctl((size_t)g.Cg * d.R * d.S);
    for (size_t col = 0; col < ctl.size(); ++col) {
        const int s = (int)(col % d.S), r = (int)(col / d.S % d.R), cl = (int)(col / ((size_t)d.R * d.S)), tap = r * d.S + s;
        const int at = row_seen[r] && col_seen[s] ? r * d.W + s : 0;
        ctl[col] = (uint32_t)(cl * d.H * d.W + at) * 4u << 3 | (uint32_t)(four ? tap : 31 - tap);
    }
    // padding: weight 0 on a tap no position has (the four-position kernel reads there: channel 1, inside the tensor)
    const uint64_t pad_entry = four ? (uint64_t)((uint32_t)(d.H * d.W) * 4u << 3 | 31u) << 32 : 0;
    const int last = (g.Cg - 1) * d.R * d.S;       // first column of a group's last channel
    std::vector<uint64_t> edge;
    for (int k = 0; k < d.K; ++k) {
        const int grp = k / g.Kg;
        const uint32_t add = (uint32_t)(grp * g.Cg * d.H * d.W) * 4u << 3;
        const size_t start = out.ent.size();
        edge.clear();
        for (int j = c.rowptr[k]; j < c.rowptr[k + 1]; ++j) {
            const int col = c.colidx[j];
            uint32_t vb;
            std::memcpy(&vb, &c.val[j], 4);
            const uint64_t e = (uint64_t)vb | (uint64_t)(ctl[col] + add) << 32;
            if (four && ((grp == 0 && col < d.R * d.S) || (grp == d.groups - 1 && col >= last)))
                edge.push_back(e);
            else
                out.ent.push_back(e);
        }
        while ((out.ent.size() - start) % SCONV_GATHER_CHUNK) out.ent.push_back(pad_entry);
        if (four) {
            out.rowptr[3 * (size_t)k] = (int32_t)start;
            out.rowptr[3 * (size_t)k + 1] = (int32_t)((out.ent.size() - start) / SCONV_GATHER_CHUNK);
            out.rowptr[3 * (size_t)k + 2] = (int32_t)edge.size();
            out.ent.insert(out.ent.end(), edge.begin(), edge.end());
        } else {
            out.rowptr[k + 1] = (int32_t)out.ent.size();
        }
        if (out.ent.size() >= ((size_t)1 << 30)) return SCONV_ERR_RANGE;
    }
    out.ent.resize(out.ent.size() + SCONV_GATHER_CHUNK, 0); // the kernel reads one chunk ahead
    return SCONV_OK;
}

int pack_fc_gather(const sconv_desc &d, const Canonical &c, PackedGather &out)
{
    out.rowptr = c.rowptr;
    out.ent.resize(c.val.size());
    for (size_t j = 0; j < c.val.size(); ++j) {
        uint32_t vb;
        std::memcpy(&vb, &c.val[j], 4);
        out.ent[j] = (uint64_t)vb | ((uint64_t)(uint32_t)c.off[j] << 32); // 1x1 image: the offset is the feature
    }
    return SCONV_OK;
}

// The kernel's own limits: a tap per bit of the lane mask, the image's byte offsets in 29 bits, everything else in 31.
bool gather_fits(const sconv_desc &d, int N)
{
    const Geometry g = geometry(d);
    const int64_t HW = (int64_t)d.H * d.W, OHW = (int64_t)g.OH * g.OW;
    if ((int64_t)d.R * d.S > SCONV_GATHER_MAX_TAPS) return false;
    if ((d.C * HW + ((int64_t)d.R * d.W + d.S)) * 4 >= ((int64_t)1 << 29)) return false;
    return (int64_t)N * d.C * HW * 4 < ((int64_t)1 << 30) && (int64_t)N * OHW < ((int64_t)1 << 28) &&
           ((int64_t)d.pad * d.W + d.pad) * 4 < ((int64_t)1 << 28);
}

bool fc_gather_fits(const sconv_desc &d, int N)
{
    return N >= 4 && N % 4 == 0 && N <= SCONV_FC_GATHER_MAX_N && (int64_t)d.C * N * 4 < ((int64_t)1 << 32);
}

// What a gather launch takes, in microseconds: 3 us whatever it does, then the longer of two terms and a third of the
// shorter one.  Throughput: a wave's index arithmetic and a 64-lane load have a price each; latency: a wave's chunks of 8
// nonzeros follow each other, the longest row counts.  Fitted for the four-position kernel to 60 random layers (3-85 us,
// 14 % off on average): 0.25 us per thousand waves, 29 us per million loads (of 256 positions), 0.35 us per chunk; for the
// other one to 37 (0.1-480 million multiply-adds): 0.12 us (30 % more for a second chunk of positions), 18 us per million
// loads of 64 positions (25 % more when the lanes are a stride apart), 0.28 us.
GatherShape choose_gather(const sconv_desc &d, int N, double avg_row_nnz, int max_row_nnz)
{
    const Geometry g = geometry(d);
    const bool four = gather4_fits(d);
    const double P = four ? (double)N * g.OH * ceil_div(g.OW, 4) : (double)N * g.OH * g.OW; // (counted through the image they are fewer: up to a fifth less)
    GatherShape best = {0, 0, 0.0, 0.0, 0.0};
    for (int t = 1; t <= (four ? 1 : 2); ++t)
        for (int split = 1; split <= 8; split *= 2) {
            const double tiles = std::ceil(P / (64.0 * t)), chunks = std::max(1.0, std::ceil(avg_row_nnz / SCONV_GATHER_CHUNK + 0.4));
            const double waves = d.K * tiles * split, chunks_wave = std::ceil((double)max_row_nnz / (SCONV_GATHER_CHUNK * split));
            double loads = d.K * tiles * t * chunks * SCONV_GATHER_CHUNK, thr, lat;
            if (four) {
                loads += d.K * tiles * 8.0 * avg_row_nnz / d.C;          // entries of the two outer channels: four loads each
                thr = 0.25e-3 * waves + 0.029e-3 * loads;
                lat = 0.35 * chunks_wave;
            } else {
                thr = 0.12e-3 * waves * (1.0 + 0.3 * (t - 1)) + 0.018e-3 * loads * (d.stride > 1 ? 1.25 : 1.0);
                lat = 0.28 * chunks_wave * std::sqrt((double)t);
            }
            const double us = 3.0 + std::max(thr, lat) + 0.35 * std::min(thr, lat);
            if (best.t == 0 || us < best.us) best = GatherShape{t, split, us, 1.25, 0.0};
        }
    // 1.25 (of 260 random calls 2 then come here wrongly by more than 2 % and 16 stay away wrongly by more than 5 %; 5 and 9 at
    // 1.15), and more where the model reads low.  19953 random calls that it sent to these kernels were timed in turn against the flat-stream
    // kernel: 298 took more than 2 % longer, 92 more than 20 %, most of them in two places.
    // A row much longer than the others, whose waves walk more than eight chunks: they share their CU with the waves of other
    // rows and take longer over a chunk than alone, and start last as often as first.
    // A few workgroups more than there are CUs: the CUs that get a second one are done last.
    // With the larger factors there 176 and 41 are left (7074 of the calls had no part in choosing them: 31 of more than 20 %
    // before, 15 after), and the 276 calls that change kernel take as long in sum.
    if (best.t > 0) {
        const int rows = best.split >= 4 ? 1 : 4 / best.split;
        const double tiles = std::ceil(P / (64.0 * best.t)), wgs = tiles * ceil_div(d.K, rows);
        if (max_row_nnz >= 3.0 * avg_row_nnz + SCONV_GATHER_CHUNK && ceil_div(max_row_nnz, SCONV_GATHER_CHUNK * best.split) > 8) best.margin = 1.5;
        // (By rows also where the fours are counted through the image, which leaves fewer workgroups: 216 -> 35, 18x18, batch 5, 280 and 245 of
        // them, stays at 24.3 us and would take 15.1.)
        if (wgs > 256 && wgs < 320) best.margin = 1.75;
        // Against the flat streams on the vector units the four-position kernel is trusted further where its rows are level and the launch
        // is short (the input then comes from L2), and its model reads high where output rows leave fours partly empty: what fours through the
        // image would take counts, however they are counted (50 random calls that this brings 1.19x, 5 of them more than 2 % slower).  Of
        // 996 random calls that moved there at 1.08 50 were more than 2 % slower, down to 0.77x (1.24x on average), of 161 of a later draw 6, down
        // to 0.74x (1.28x); their sums are half as far from the exact ones.  Not taken: to leave out long rows of several taps over more than
        // 20 MB (15 of 35 calls slower on the gather kernel, 1.01x on average, 6 of 21 of another draw, 1.02x), rows over eight waves (3 of 4; 1 of
        // 5, 1.03x).  384 -> 256 in two groups, 13x13, batch 16, density 0.1: 25.3 -> 22.7 us.  (Skewed rows: down to 0.59x, strided layers to
        // 0.74x, long launches to 0.81x.  Against the matrix cores 1.25 stays: 40 of 42 such calls were slower on the gather kernel, 0.68x.)
        if (four && best.margin == 1.25 && max_row_nnz < 2.0 * avg_row_nnz + SCONV_GATHER_CHUNK && best.us <= 40.0) {
            const double by_image = g.OW == d.W && g.OW >= 4 ? std::ceil((double)N * ceil_div(g.OH * g.OW, 4) / 64.0) / tiles : 1.0;
            best.flat_us = 1.08 * (3.0 + (best.us - 3.0) * by_image);
        }
    }
    return best;
}

// The same for the fully connected kernel; t is the number of lanes (16-byte pieces of the batch) that share a nonzero.
// A load instruction costs 50 us per million and up to 230 us more, the more separate pieces of memory its lanes read
// (64 / t); a round of four nonzeros per lane group takes 0.28 us of latency.
GatherShape choose_fc_gather(const sconv_desc &d, int N, double avg_row_nnz, int max_row_nnz)
{
    const int n4 = N / 4;
    GatherShape best = {0, 0, 0.0, 0.0, 0.0};
    for (int t = 1; t <= 32 && t < 2 * n4; t *= 2)
        for (int split = 1; split <= 16; split *= 4) {
            const double per_round = 4.0 * (64 / t) * split;
            const double waves = (double)d.K * split * std::ceil((double)n4 / t);
            const double rounds = std::max(1.0, std::ceil(avg_row_nnz / per_round + 0.3));
            const double thr = 0.03e-3 * waves + (0.05e-3 + 0.23e-3 / t) * waves * rounds * 4.0;
            const double lat = 0.28 * std::ceil(max_row_nnz / per_round);
            const double us = 2.9 + std::max(thr, lat) + 0.35 * std::min(thr, lat);
            if (best.t == 0 || us < best.us) best = GatherShape{t, split, us, 1.2, 0.0};
        }
    // Workgroups of 16 waves with long pieces of memory per nonzero, more of them than CUs: the model reads 30-40 % low.  Of 9809
    // random calls timed in turn against the flat-stream kernel 25 took more than 5 % longer with 1.2, 6 do with 1.5 here.
    if (best.split == 16 && best.t >= 16 && d.K * std::ceil((double)n4 / best.t) > 256) best.margin = 1.5;
    return best;
}

// ------------------------------------------------------------------ matrix-core kernel (rather dense layers)

bool mfma_fits(const sconv_desc &d, int N, bool feature_major)
{
    const Geometry g = geometry(d);
    const int64_t HW = (int64_t)d.H * d.W, OHW = (int64_t)g.OH * g.OW, lim = (int64_t)1 << 31;
    if ((int64_t)N * OHW >= ((int64_t)1 << 28)) return false;
    if (feature_major) return (int64_t)d.C * N * 4 < lim;
    // a workgroup's images (256 positions), from the first one's channel 0
    return (256 / OHW + 3) * d.C * HW * 4 < lim && (int64_t)g.Kg * OHW < lim;
}

// Zero, or a magnitude in [2^-94, 2^127): three bf16 parts hold it exactly, divided by SCONV_MFMA_SCALE.
bool mfma_weight_ok(float v)
{
    uint32_t u;
    std::memcpy(&u, &v, 4);
    u &= 0x7fffffffu;
    return u == 0 || (u >= 0x10800000u && u < 0x7f000000u);
}

static uint16_t to_bf16(float v) // round to nearest even
{
    uint32_t u;
    std::memcpy(&u, &v, 4);
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

static float from_bf16(uint16_t b)
{
    const uint32_t u = (uint32_t)b << 16;
    float v;
    std::memcpy(&v, &u, 4);
    return v;
}

// A 1x1 layer sees its image as one column: the cells a workgroup stages are then exactly its positions, not whole rows.
sconv_desc mfma_desc(const sconv_desc &d)
{
    sconv_desc f = d;
    if (d.R == 1 && d.S == 1 && d.stride == 1 && d.pad == 0) {
        f.H = d.H * d.W;
        f.W = 1;
    }
    return f;
}

bool choose_mfma(const sconv_desc &layer, int N, MfmaTiling &t)
{
    const sconv_desc d = mfma_desc(layer);
    const Geometry g = geometry(d);
    double best_units = -1;
    // an unpadded strided layer may be seen as its phase images: fewer empty channels of an octet where C is small
    for (int phased = 0; phased <= (d.stride > 1 && d.pad == 0 ? 1 : 0); ++phased) {
        MfmaTiling c;
        const int s = phased ? d.stride : 1;
        c.phased = phased != 0;
        c.cstep = s;
        c.lstep = phased ? 1 : d.stride;
        c.Rr = ceil_div(d.R, s);
        c.Sr = ceil_div(d.S, s);
        if ((int64_t)g.Cg * s * s > (1 << 20) || (int64_t)(g.OW - 1) * c.lstep + c.Sr > 1024) continue;
        c.c_virtual = g.Cg * s * s;
        c.Wl = (g.OW - 1) * c.lstep + c.Sr;
        // rows of cells that 256 (or 128) consecutive positions touch, over all places they can start at
        auto cells_of = [&](int bn) {
            const int rows_out = ceil_div(bn - 1, g.OW) + 1, images = c.Rr > c.lstep ? ceil_div(bn - 1, g.OH * g.OW) + 1 : 1;
            return ((int64_t)rows_out * c.lstep + (int64_t)images * (c.Rr - c.lstep)) * c.Wl;
        };
        // (layers of one tap are a few matrix steps per staged channel: they want deep blocks, and 128 positions leave LDS
        // for twice the octets; 192 -> 64 on 28x28, batch 64: 6 blocks of 4 octets 25 us, 2 of 12 22 us)
        c.nt_max = cells_of(256) <= 1024 && c.Rr * c.Sr > 1 ? 2 : 1;
        const int64_t cells = cells_of(128 * c.nt_max);
        if (cells < 1 || cells > 1024) continue;
        c.plane = (int)((cells + 63) / 64 * 64);
        const int taps = c.Rr * c.Sr, octets = ceil_div(c.c_virtual, 8);
        c.one_tap = taps == 1 && c.cstep == 1 && c.lstep == 1 && c.Wl == 1 && d.pad == 0 && (128 / ((int64_t)g.OH * g.OW) + 1) * d.K * g.OH * g.OW * 4 < ((int64_t)1 << 31);
        for (int g8 = 1; g8 <= std::min(octets, 16); ++g8) {
            c.g8 = g8;
            c.nblk = ceil_div(octets, g8);
            c.steps = ceil_div(taps * g8, 2);
            c.steps_last = ceil_div(taps * (octets - (c.nblk - 1) * g8), 2);
            const int64_t lds = (int64_t)g8 * c.plane * 48 + 8 * (c.steps + c.steps_last) + 4 * c.plane;
            if (lds > 80 * 1024 - 256) break;                 // two workgroups on a CU
            const int64_t total = (int64_t)(c.nblk - 1) * c.steps + c.steps_last;
            if (total > (1 << 18)) continue;
            c.total_steps = (int)total;
            c.lds_bytes = (int)lds;
            const double units = total + 1.0 * c.nblk;        // a block's barriers and first reads weigh about a step
            if (best_units < 0 || units < best_units) {
                best_units = units;
                t = c;
            }
        }
    }
    if (best_units < 0) return false;
    t.n_tiles32 = 2 * ceil_div(g.Kg, 64);
    // What a launch takes, fitted to 26 layers in every shape and checked on 50 more (10-460 us, 12 % off on average): a
    // workgroup's matrix instructions at 2.1 GHz, 0.61 us for each round of 64 cells x 8 channels x 4 waves it stages, 4 us
    // for its index arithmetic; workgroups that share a CU overlap down to 1.3 times the first and half of the others; the
    // output at 6 TB/s, stored when a workgroup is done.
    t.us = 0;
    const double P = (double)N * g.OH * g.OW, out_bytes = 4.0 * P * d.K;
    for (int mt = 1; mt <= 2; ++mt)
        for (int nt = 1; nt <= t.nt_max; ++nt)
            for (int splits : {1, 2, 3, 4, 6, 8, 12, 16}) {
                if (splits > t.nblk || ceil_div(t.nblk, ceil_div(t.nblk, splits)) != splits) continue;
                if (splits > 1 && out_bytes * splits > SCONV_NOALLOC_SCRATCH_BYTES) continue;
                const int n_mtiles = ceil_div(g.Kg, 32 * mt), blocks = ceil_div(t.nblk, splits);
                const double wgs = std::ceil(P / (128.0 * nt)) * n_mtiles * d.groups * splits, per_cu = std::ceil(wgs / 256.0);
                const double share = (double)blocks / t.nblk;
                const double mfma = share * t.total_steps * mt * nt * 192.0 / 2100.0;
                const double rounds = blocks * std::ceil(t.plane * (nt == t.nt_max ? 1.0 : 0.6) / 64.0) * t.g8 / 4.0;
                const int fit = std::min(mt * nt == 4 ? 2 : mt * nt == 2 ? 3 : 4, 160 * 1024 / (t.lds_bytes + 512));
                const double alone = mfma + 0.05 * blocks + 0.61 * rounds + 4.0, shared = mfma / 0.78 + 0.306 * rounds + 1.2;
                double us = 4.4 + std::max(alone * std::ceil(per_cu / fit), per_cu * shared) + out_bytes / 6.0e6;
                // partial sums: stored, and added by a launch of their own that reads every part
                if (splits > 1) us += 4.0 + splits * (out_bytes / 3.5e6 + 0.3);
                if (t.us == 0 || us < t.us) {
                    t.us = us;
                    t.mt = mt;
                    t.nt = nt;
                    t.splits = splits;
                    t.n_mtiles = n_mtiles;
                }
            }
    return true;
}

bool choose_mfma_column(const sconv_desc &d, int N, int min_splits, MfmaTiling &t)
{
    const Geometry g = geometry(d);
    const double P = (double)N * g.OH * g.OW, in_bytes = 4.0 * P * d.C, out_bytes = 4.0 * P * d.K;
    t.column = true;
    t.nt = 1;
    t.us = 0;
    // Blocks of whole steps of 16 channels, of the size that leaves the fewest (parts are whole blocks; LDS holds one only where sums
    // are taken again).
    const int octets = ceil_div(g.Cg, 8);
    double best_units = -1;
    for (int g8 = 1; g8 <= std::min(octets, 16); ++g8) {
        const int64_t lds = (int64_t)g8 * t.plane * 48 + 16 * ceil_div(g8, 2) + 4 * t.plane;
        if ((g8 % 2 && g8 < octets) || lds > 80 * 1024 - 256) continue;
        const int nblk = ceil_div(octets, g8), steps = ceil_div(g8, 2), steps_last = ceil_div(octets - (nblk - 1) * g8, 2), total = (nblk - 1) * steps + steps_last;
        if (best_units >= 0 && total + nblk >= best_units) continue;
        best_units = total + nblk;
        t.g8 = g8;
        t.nblk = nblk;
        t.steps = steps;
        t.steps_last = steps_last;
        t.total_steps = total;
        t.lds_bytes = (int)lds;
    }
    // Fitted to 110 random layers in every shape (646 launches of 5-200 us, 4 % off on average, 26 % at most, low where there are few
    // steps and many filters): a step of a workgroup on its CU, its head and stores; the input from memory; the output.  32 filters count
    // 1.05 times: the shape chosen then takes 0.9 % longer than the best one on average, 15 % at most.
    for (int mt = 1; mt <= 2; ++mt)
        for (int splits : {1, 2, 3, 4, 6, 8, 12, 16}) {
            if (splits < min_splits || splits > t.nblk || ceil_div(t.nblk, ceil_div(t.nblk, splits)) != splits) continue;
            if (splits > 1 && out_bytes * splits > SCONV_NOALLOC_SCRATCH_BYTES) continue;
            const int n_mtiles = ceil_div(g.Kg, 32 * mt);
            const double per_cu = std::ceil(std::ceil(P / 128.0) * n_mtiles * d.groups * splits / 256.0);
            const double steps = std::min(t.total_steps, ceil_div(t.nblk, splits) * t.steps);
            double us = 5.0 + std::max(per_cu * (mt == 1 ? 0.216 * steps + 0.32 : 0.293 * steps + 0.86), in_bytes / 5.0e6);
            us += splits > 1 ? 1.45 + splits * (out_bytes / 2.5e6 + 0.24) : out_bytes / 4.6e6;
            if (mt == 1) us *= 1.05;
            if (t.us == 0 || us < t.us) {
                t.us = us;
                t.mt = mt;
                t.splits = splits;
                t.n_mtiles = n_mtiles;
            }
        }
    return t.us > 0;
}

int pack_mfma(const sconv_desc &d, const Canonical &c, const MfmaTiling &t, PackedMfma &out)
{
    const Geometry g = geometry(d);
    const int s = t.phased ? d.stride : 1, taps = t.Rr * t.Sr, octets = ceil_div(t.c_virtual, 8);
    const int g8_last = octets - (t.nblk - 1) * t.g8;
    const size_t tile_halves = (size_t)t.total_steps * 3 * 64 * 8;
    out.wfrag.assign((size_t)d.groups * t.n_tiles32 * tile_halves + 3 * 64 * 8, 0); // the kernel reads one step ahead
    // where a column's weight of row 0 goes inside a 32-row tile
    std::vector<uint32_t> at_col((size_t)g.Cg * d.R * d.S);
    for (size_t col = 0; col < at_col.size(); ++col) {
        const int fs = (int)(col % d.S), fr = (int)(col / d.S % d.R), cl = (int)(col / ((size_t)d.R * d.S));
        const int cv = t.phased ? ((fr % s) * s + fs % s) * g.Cg + cl : cl;
        const int tap = (fr / s) * t.Sr + fs / s, oct = cv / 8, b = oct / t.g8, ol = oct - b * t.g8;
        const int u = tap * (b == t.nblk - 1 ? g8_last : t.g8) + ol;
        at_col[col] = (uint32_t)(((size_t)(b * t.steps + u / 2) * 3 * 64 + 32 * (u % 2)) * 8 + cv % 8);
    }
    for (int k = 0; k < d.K; ++k) {
        const int grp = k / g.Kg, kl = k - grp * g.Kg;
        uint16_t *tile = &out.wfrag[((size_t)grp * t.n_tiles32 + kl / 32) * tile_halves + (size_t)(kl % 32) * 8];
        for (int j = c.rowptr[k]; j < c.rowptr[k + 1]; ++j) {
            if (!mfma_weight_ok(c.val[j])) return SCONV_ERR_PLAN;
            const float v = c.val[j] / SCONV_MFMA_SCALE;
            const uint16_t h = v == 0.f ? 0x8000 : to_bf16(v);
            const float r1 = v - from_bf16(h);
            const uint16_t m = to_bf16(r1);
            uint16_t *at = tile + at_col[c.colidx[j]];
            at[0] = h;
            at[64 * 8] = m;
            at[2 * 64 * 8] = to_bf16(r1 - from_bf16(m));
        }
    }
    out.uoff.assign((size_t)2 * (t.steps + t.steps_last), 0);
    for (int last = 0; last < 2; ++last) {
        const int g8 = last ? g8_last : t.g8;
        for (int tap = 0; tap < taps; ++tap)
            for (int ol = 0; ol < g8; ++ol)
                out.uoff[(last ? 2 * t.steps : 0) + tap * g8 + ol] = (ol * t.plane + (tap / t.Sr) * t.Wl + tap % t.Sr) * 48;
    }
    // (a phase no filter tap falls into is nothing but zeros in the weights; its first element may lie past the input)
    out.choff.clear();
    if (t.phased)
        for (int cv = 0; cv < octets * 8; ++cv) {
            const int ph = cv / g.Cg, cl = cv % g.Cg;
            const bool there = cv < t.c_virtual && ph / s < d.R && ph % s < d.S;
            out.choff.push_back(there ? ((cl * d.H + ph / s) * d.W + ph % s) * 4 : SCONV_MFMA_NO_CHANNEL);
        }
    return SCONV_OK;
}

// ------------------------------------------------------------------ flat streams on the matrix cores

// How often a step's octet is needed, on average over the workgroups (the waves of one wait for each other): once where one of a wave's row tiles has weights in it, twice
// where a row has more than two of four channels.  The second time of a few tiles goes to steps of their own (an octet per tile),
// of many tiles to the shared steps.  Rows as pack_flat_mc orders them, their weights taken as evenly spread.
static double mc_slots_per_octet(const sconv_desc &d, const Canonical &c, int mt, int wr)
{
    const Geometry g = geometry(d);
    const double cols = (double)g.Cg * d.R * d.S;
    std::vector<int> nnz(g.Kg);
    double sum = 0;
    int units = 0;
    for (int grp = 0; grp < d.groups; ++grp) {
        for (int k = 0; k < g.Kg; ++k) nnz[k] = c.rowptr[grp * g.Kg + k + 1] - c.rowptr[grp * g.Kg + k];
        std::sort(nnz.begin(), nnz.end(), std::greater<int>());
        double most = 0;
        for (int r0 = 0, u = 0; r0 < g.Kg; r0 += 16 * mt, ++u) {
            double none = 1, once = 1, tiles = 0;       // no row has weights in an octet, no row needs it twice, tiles that do
            for (int t0 = r0; t0 < std::min(g.Kg, r0 + 16 * mt); t0 += 16) {
                double tile = 1;
                for (int r = t0; r < std::min(g.Kg, t0 + 16); ++r) {
                    const double x = std::min(1.0, nnz[r] / cols), q = 4 * x * x * x * (1 - x) + x * x * x * x;
                    none *= std::pow(1 - x, 8);
                    tile *= (1 - q) * (1 - q);
                }
                once *= tile;
                tiles += 1 - tile;
            }
            most = std::max(most, 1 - none + std::min(1 - once, 1.5 * tiles / mt));
            if (u % wr == wr - 1 || r0 + 16 * mt >= g.Kg) {
                sum += most;
                most = 0;
                ++units;
            }
        }
    }
    return sum / std::max(1, units);
}

int shortest_row(const Canonical &c)
{
    int shortest = 0;
    for (size_t k = 1; k < c.rowptr.size(); ++k) {
        const int nnz = c.rowptr[k] - c.rowptr[k - 1];
        if (nnz > 0 && (shortest == 0 || nnz < shortest)) shortest = nnz;
    }
    return shortest;
}

bool flat_mc_weights_ok(const sconv_desc &d, const Canonical &c)
{
    if ((double)c.val.size() < (double)SCONV_MC_FLUSHED_ROW * d.K || shortest_row(c) < SCONV_MC_FLUSHED_ROW) return false;
    float most = 0, least = INFINITY;
    for (float v : c.val) {
        const float m = std::fabs(v);
        most = std::max(most, m);
        if (!(m <= 3.4028235e38f)) return false;
        if (m > 0) least = std::min(least, m);
    }
    return most == 0 || (most >= 0x1p-100f && most <= 0x1p100f && least >= most * 0x1p-26f);
}

bool choose_flat_mc(const sconv_desc &layer, const Canonical &csr, int N, bool flushed, FlatMcTiling &t)
{
    const double avg_row_nnz = (double)csr.val.size() / std::max(1, layer.K);
    if (avg_row_nnz < SCONV_MC_FLUSHED_ROW) return false;
    const sconv_desc d = mfma_desc(layer);
    const Geometry g = geometry(d);
    const double density = std::min(1.0, avg_row_nnz / ((double)g.Cg * d.R * d.S));
    if (d.H * d.W > 1 && (256 / ((int64_t)g.OH * g.OW) + 3) * d.K * g.OH * g.OW * 4 >= ((int64_t)1 << 31)) return false; // 32-bit store offsets
    // Rather dense layers (most octets twice): 64 filters x 128 positions, the sums flushed every few steps.  The others: up to
    // 128 x 128.  As few padded filters as possible, rather more than fewer.
    const bool dense = density >= SCONV_MC_DENSE;
    int mt = 0, wr = 0;
    double best_rows = 0;
    const int shapes[][2] = {{4, 2}, {3, 2}, {4, 1}, {3, 1}, {2, 1}};
    for (const auto &sh : shapes) {
        if (dense && sh[1] == 2) continue;
        const int rows = 16 * sh[0] * sh[1];
        const double cost = (double)ceil_div(g.Kg, rows) * rows * (sh[0] == 4 ? 1.0 : sh[0] == 3 ? 1.06 : 1.2) * (sh[1] == 2 ? 1.0 : 1.1);
        if (mt == 0 || cost < best_rows) {
            best_rows = cost;
            mt = sh[0];
            wr = sh[1];
        }
    }
    const int pos_waves = wr == 2 ? 2 : 4;
    const double slots = mc_slots_per_octet(d, csr, mt, wr);
    double best_units = -1, steps_total = 0, rows_at[2] = {0, 0};
    for (int phased = 0; phased <= (d.stride > 1 && d.pad == 0 ? 1 : 0); ++phased) {
        FlatMcTiling c;
        const int s = phased ? d.stride : 1;
        c.phased = phased != 0;
        c.runs = phased && s % 4 == 0 && d.S >= s;
        c.cstep = s;
        c.lstep = phased ? 1 : d.stride;
        c.Rr = ceil_div(d.R, s);
        c.Sr = ceil_div(d.S, s);
        if ((int64_t)g.Cg * s * s > (1 << 20) || (int64_t)(g.OW - 1) * c.lstep + c.Sr > 1024) continue;
        c.c_virtual = g.Cg * s * s;
        c.Wl = (g.OW - 1) * c.lstep + c.Sr;
        // the right padding of a row is the left padding of what follows it
        int over = 0;
        if (d.stride == 1 && d.W + d.pad >= g.OW && c.Wl > d.W + d.pad) {
            over = c.Wl - (d.W + d.pad);
            c.Wl = d.W + d.pad;
        }
        if (over > d.pad) continue;
        // rows that a workgroup's consecutive positions touch, over all places they can start at
        auto rows_of = [&](int bn) {
            const int rows_out = ceil_div(bn - 1, g.OW) + 1, images = c.Rr > c.lstep ? ceil_div(bn - 1, g.OH * g.OW) + 1 : 1;
            return (int64_t)rows_out * c.lstep + (int64_t)images * (c.Rr - c.lstep);
        };
        c.nt_max = !dense && rows_of(64 * pos_waves) * c.Wl <= 1024 ? 4 : 2;
        const int64_t n_rows = rows_of(16 * pos_waves * c.nt_max), cells = n_rows * c.Wl;
        if (cells < 1 || cells > 1024) continue;
        c.plane = (int)((cells + 63) / 64 * 64);
        // Sixteen lanes read sixteen consecutive positions: without bank conflicts also across the end of a row if the pitch is
        // as many units as there are positions in a row, modulo 16.  High and low parts of a row side by side leave little room
        // unused then; where they would leave much, they go to planes of their own.
        c.pitch = 2 * c.Wl + ((g.OW * c.lstep - 2 * c.Wl) % 16 + 16) % 16;
        c.part = c.Wl;
        c.octet = (int)(n_rows * c.pitch + over);
        if (g.OW == 1 || c.pitch * 8 > c.Wl * 19) {
            c.pitch = c.Wl;
            c.part = (int)(n_rows * c.pitch + over);
            c.octet = 2 * c.part;
        }
        c.octet = (c.octet + 15) / 16 * 16; // lanes of two quarters are served together: their octets at one tap must not collide
        const int taps = c.Rr * c.Sr, octets = ceil_div(c.c_virtual, 8);
        for (int g8 = 1; g8 <= std::min(octets, 32); ++g8) {
            c.g8 = g8;
            c.nblk = ceil_div(octets, g8);
            if (g8 != ceil_div(octets, c.nblk)) continue;     // blocks alike
            const int64_t lds = std::max<int64_t>((int64_t)g8 * c.octet * 16 + 8 * c.plane, 4 * SCONV_MC_STORE_BYTES(mt, c.nt_max)) + 16;
            if (lds > 80 * 1024 - 256 || (int64_t)g8 * taps * 2 > 0xffff) break; // two workgroups on a CU
            c.lds_bytes = (int)lds;
            auto steps_of = [&](int o) { return std::max<double>(ceil_div(taps * o, 8), taps * o * slots / 8 + 0.5); };
            const double steps = (c.nblk - 1) * steps_of(g8) + steps_of(octets - (c.nblk - 1) * g8);
            const double units = steps + 1.0 * c.nblk;        // a block's barriers and first reads weigh about a step
            if (best_units < 0 || units < best_units) {
                best_units = units;
                steps_total = steps;
                rows_at[0] = (double)rows_of(32 * pos_waves);
                rows_at[1] = (double)rows_of(64 * pos_waves);
                t = c;
            }
        }
    }
    if (best_units < 0) return false;
    t.mt = mt;
    t.wr = wr;
    t.n_units = ceil_div(g.Kg, 16 * mt * wr) * wr;
    t.wexp = 0;
    t.small_sum = 0;
    t.stream_bytes = 0;
    t.us = 0;
    const double P = (double)N * g.OH * g.OW, out_bytes = 4.0 * P * d.K;
    // (fitted to 60 layers of all shapes, 11-500 us: 9 % off)
    const bool wide = t.cstep == 1 && (d.W >= 4 ? t.Wl >= d.W + d.pad : t.Wl == 1 && g.OH % 4 == 0);
    const bool totals = flushed || shortest_row(csr) < SCONV_MC_ROW;
    for (int nt = 2; nt <= t.nt_max; nt += 2)
        for (int splits : {1, 2, 3, 4, 6, 8, 12, 16}) {
            if (totals && !SCONV_MC_TOTALS(mt, nt)) continue;
            if (splits > t.nblk || ceil_div(t.nblk, ceil_div(t.nblk, splits)) != splits) continue;
            if (splits > 1 && out_bytes * splits > SCONV_NOALLOC_SCRATCH_BYTES) continue;
            const int blocks = ceil_div(t.nblk, splits), positions = 16 * nt * pos_waves;
            const double wgs = std::ceil(P / positions) * (t.n_units / wr) * d.groups * splits, per_cu = wgs / 256.0;
            // (a column that is read feeds half as many products with two row tiles as with four; with two of columns as well that is
            // not hidden: 12 layers took 1.07-1.5 times what they were read as, the longer the more, the other shapes 0.8-1.2)
            const double steps = (double)blocks / t.nblk * steps_total * mt * nt * (mt == 2 && nt == 2 ? 1.45 : 1.0), stored = 16.0 * mt * wr * positions * 4 / 6900.0;
            const double cells = blocks * rows_at[nt / 2 - 1] * t.Wl * std::min(t.g8, ceil_div(t.c_virtual, 8));
            const double stage = 0.66 * blocks + cells * (wide ? 0.00086 : 0.0018);
            const double two = 3.3 + stage + steps * (nt == 4 ? 0.080 : 0.092) + stored;     // workgroups on a CU
            const double one = 3.3 + 1.4 * stage + steps * 0.056 + 0.3 * stored;
            double us = 3.8;
            if (per_cu <= 1) us += one;
            else if (per_cu <= 2) us += two;
            else us += two * (per_cu > 4 ? 1 + 0.98 * (per_cu / 2 - 1) : 1 + 1.07 * (std::ceil(per_cu) / 2 - 1));
            if (splits > 1) us += 2.0 + splits * (out_bytes / 1.7e6);
            if (t.us == 0 || us < t.us) {
                t.us = us;
                t.nt = nt;
                t.splits = splits;
            }
        }
    return true;
}

static uint16_t to_f16(float v) // round to nearest even; |v| below 65520, denormals carried
{
    uint32_t u;
    std::memcpy(&u, &v, 4);
    const uint16_t sign = (uint16_t)(u >> 16 & 0x8000u);
    u &= 0x7fffffffu;
    if (u < 0x38800000u) { // below 2^-14: adding 2^-1 leaves the value's multiple of 2^-24 in the low bits
        float m;
        std::memcpy(&m, &u, 4);
        m += 0.5f;
        std::memcpy(&u, &m, 4);
        return (uint16_t)(sign | (uint16_t)(u - 0x3f000000u));
    }
    u += 0xfffu + (u >> 13 & 1u);
    return (uint16_t)(sign | (uint16_t)((u >> 13) - (112u << 10)));
}

static float from_f16(uint16_t b)
{
    uint32_t u = (uint32_t)(b & 0x7fffu) << 13;
    float v;
    std::memcpy(&v, &u, 4);
    v *= 0x1p112f;
    return b & 0x8000u ? -v : v;
}

// Which of four channels a row's nth use of them takes (two at most, in order; the places of what is not real only differ).
struct Pick {
    uint8_t at[2], real[2], places;
};
static const struct Picks {
    Pick pick[2][16];
    uint8_t uses[256]; // of an octet by a row that has these of its channels
    Picks()
    {
        for (int both = 0; both < 256; ++both) {
            const int most = std::max(__builtin_popcount(both & 15), __builtin_popcount(both >> 4));
            uses[both] = (uint8_t)((most + 1) / 2);
        }
        for (int nth = 0; nth < 2; ++nth)
            for (int four = 0; four < 16; ++four) {
                Pick &p = pick[nth][four];
                int ch[4], n = 0;
                for (int z = 0; z < 4; ++z)
                    if (four >> z & 1) ch[n++] = z;
                p = {{0, 1}, {0, 0}, 0};
                const int left = std::min(2, n - 2 * nth);
                if (left == 2) {
                    p = {{(uint8_t)ch[2 * nth], (uint8_t)ch[2 * nth + 1]}, {1, 1}, 0};
                } else if (left == 1) {
                    const int z = ch[2 * nth];
                    p = z == 3 ? Pick{{0, 3}, {0, 1}, 0} : Pick{{(uint8_t)z, 3}, {1, 0}, 0};
                }
                p.places = (uint8_t)(p.at[0] | p.at[1] << 2);
            }
    }
} kPicks;

int pack_flat_mc(const sconv_desc &layer, const Canonical &c, FlatMcTiling &t, PackedFlatMc &out)
{
    const sconv_desc &d = layer;
    const Geometry g = geometry(d);
    const int s = t.phased ? d.stride : 1, taps = t.Rr * t.Sr, octets = ceil_div(t.c_virtual, 8), rows = 16 * t.mt;
    const int slots = octets * taps; // block after block, tap after tap, octet after octet
    const size_t rec = SCONV_MC_RECORD(t.mt);
    const int meta = (t.mt + 1) / 2 * 2 + 2; // 16-bit words a lane has behind the weights
    float most = 0;
    for (float v : c.val) most = std::max(most, std::fabs(v));
    int e = 0;
    std::frexp(most, &e);
    t.wexp = most > 0 ? 14 - e : 0;
    const float scale = std::ldexp(1.f, t.wexp);
    std::vector<int32_t> col_slot((size_t)g.Cg * d.R * d.S); // slot * 8 + channel of the octet
    std::vector<int32_t> slot_off(slots), block_first(t.nblk + 1);
    for (int b = 0; b <= t.nblk; ++b) block_first[b] = std::min(b * t.g8, octets) * taps;
    for (int b = 0; b < t.nblk; ++b) {
        const int o8 = std::min(t.g8, octets - b * t.g8);
        for (int tap = 0; tap < taps; ++tap)
            for (int ol = 0; ol < o8; ++ol)
                slot_off[block_first[b] + tap * o8 + ol] = ol * t.octet + (tap / t.Sr) * t.pitch + tap % t.Sr;
    }
    for (size_t col = 0; col < col_slot.size(); ++col) {
        const int fs = (int)(col % d.S), fr = (int)(col / d.S % d.R), cl = (int)(col / ((size_t)d.R * d.S));
        const int ph = (fr % s) * s + fs % s, cv = !t.phased ? cl : t.runs ? cl * s * s + ph : ph * g.Cg + cl;
        const int oct = cv / 8, b = oct / t.g8, o8 = std::min(t.g8, octets - b * t.g8);
        const int tap = (fr / s) * t.Sr + fs / s;
        col_slot[col] = (block_first[b] + tap * o8 + oct - b * t.g8) * 8 + cv % 8;
    }
    out = PackedFlatMc();
    out.seg.assign((size_t)d.groups * t.n_units * t.nblk * 2, 0);
    out.row_of.assign((size_t)d.groups * t.n_units * rows, -1);
    // rows of like length together: tiles of short rows need fewer octets twice, or at all
    std::vector<int32_t> order(d.K);
    std::iota(order.begin(), order.end(), 0);
    for (int grp = 0; grp < d.groups; ++grp)
        std::stable_sort(order.begin() + grp * g.Kg, order.begin() + (grp + 1) * g.Kg,
                         [&](int a, int b) { return c.rowptr[a + 1] - c.rowptr[a] > c.rowptr[b + 1] - c.rowptr[b]; });
    struct Item {
        int32_t slot;
        int tiles, nth;
    };
    // one wave's filters: its records, numbered from 0 until all are there
    auto pack_unit = [&](int unit, std::vector<uint8_t> &stream, double &norm) -> int {
        std::vector<uint8_t> mask((size_t)rows * slots);   // channels of an octet that a row has
        std::vector<float> val((size_t)slots * 8);         // one row's weights
        std::vector<uint8_t> need((size_t)t.mt * slots);   // how often a tile needs an octet: 0, 1, 2
        std::vector<uint8_t> shared(slots);
        std::vector<int32_t> where((size_t)(t.mt + 1) * slots * 2); // record * 8 + octet of an octet's nth use: shared, then by tile
        std::vector<Item> items[5];                        // by the number of tiles
        stream.reserve((size_t)(slots / 8 + t.nblk) * rec * 5 / 4);
        int64_t n_rec = 0;
        const int grp = unit / t.n_units, r0 = (unit - grp * t.n_units) * rows, n_rows = std::max(0, std::min(rows, g.Kg - r0));
        int32_t *row_of = &out.row_of[(size_t)unit * rows];
        for (int r = 0; r < n_rows; ++r) {
            const int k = row_of[r] = order[grp * g.Kg + r0 + r];
            uint8_t *m = &mask[(size_t)r * slots], *n = &need[(size_t)(r / 16) * slots];
            for (int j = c.rowptr[k]; j < c.rowptr[k + 1]; ++j) {
                const int at = col_slot[c.colidx[j]];
                m[at / 8] |= (uint8_t)(1u << (at & 7));
            }
            for (int i = 0; i < slots; ++i) n[i] = std::max(n[i], kPicks.uses[m[i]]);
        }
        for (int b = 0; b < t.nblk; ++b) {
            const int lo = block_first[b], hi = block_first[b + 1];
            for (auto &v : items) v.clear();
            int n_items = 0;
            for (int i = lo; i < hi; ++i) {
                shared[i] = 0;
                for (int nth = 1; nth >= 0; --nth) {
                    int tiles = 0;
                    for (int m = 0; m < t.mt; ++m) tiles += need[(size_t)m * slots + i] > nth;
                    if (tiles) items[tiles].push_back({i, tiles, nth});
                    n_items += tiles > 0;
                    shared[i] += tiles > 0;
                }
            }
            // what single tiles need goes to steps that every tile has its own octets of, as much as these hold
            auto nth_item = [&](int i) -> const Item & {
                int z = 1;
                while (i >= (int)items[z].size()) i -= (int)items[z++].size();
                return items[z][i];
            };
            int best_p = 0, best_take = 0;
            double best = ceil_div(n_items, 8);
            for (int p = 1; p <= 4 && p < best; ++p) {
                int load[4] = {0, 0, 0, 0}, take = 0;
                for (; take < n_items; ++take) {
                    const Item &it = nth_item(take);
                    bool room = it.tiles < t.mt;
                    for (int m = 0; m < t.mt; ++m) room = room && (need[(size_t)m * slots + it.slot] <= it.nth || load[m] < 8 * p);
                    if (!room) break;
                    for (int m = 0; m < t.mt; ++m) load[m] += need[(size_t)m * slots + it.slot] > it.nth;
                }
                const double cost = ceil_div(n_items - take, 8) + SCONV_MC_PRIVATE_COST * p;
                if (cost < best) {
                    best = cost;
                    best_p = p;
                    best_take = take;
                }
            }
            for (int i = 0; i < best_take; ++i) --shared[nth_item(i).slot];
            const int n_shared = ceil_div(n_items - best_take, 8);
            int32_t *seg = &out.seg[((size_t)unit * t.nblk + b) * 2];
            seg[0] = (int32_t)n_rec;
            seg[1] = n_shared | best_p << 16;
            int pos = 0, load[4] = {0, 0, 0, 0};
            for (int i = lo; i < hi; ++i) {
                for (int nth = 0; nth < shared[i]; ++nth) where[(size_t)i * 2 + nth] = (int32_t)(n_rec * 8 + pos++);
                for (int m = 0; m < t.mt; ++m)
                    for (int nth = shared[i]; nth < need[(size_t)m * slots + i]; ++nth)
                        where[((size_t)(m + 1) * slots + i) * 2 + nth] = (int32_t)((n_rec + n_shared) * 8 + load[m]++);
            }
            bool fits = pos <= 8 * n_shared;
            for (int m = 0; m < t.mt; ++m) fits = fits && load[m] <= 8 * best_p;
            if (!fits) return SCONV_ERR_PLAN;
            n_rec += n_shared + best_p;
            if (n_rec >= 0x7fffffff / 8) return SCONV_ERR_RANGE;
            // rows without weights: places 0 and 1.  Which lanes read an octet: the first four of a step are a quarter's first
            // ones, the others its second ones
            stream.resize((size_t)n_rec * rec);
            for (int i = seg[0]; i < (int)n_rec; ++i) {
                uint16_t *lanes = reinterpret_cast<uint16_t *>(&stream[(size_t)i * rec] + t.mt * 2048);
                for (int z = 0; z < 64; ++z)
                    for (int q = 0; q < meta - 2; ++q) lanes[z * meta + q] = 0x4444;
            }
            for (int i = lo; i < hi; ++i)
                for (int m = -1; m < t.mt; ++m)
                    for (int nth = m < 0 ? 0 : shared[i]; nth < (m < 0 ? shared[i] : need[(size_t)m * slots + i]); ++nth) {
                        const int at = where[((size_t)(m + 1) * slots + i) * 2 + nth], o = at % 8;
                        uint16_t *lanes = reinterpret_cast<uint16_t *>(&stream[(size_t)(at / 8) * rec] + t.mt * 2048);
                        for (int l = m < 0 ? 0 : m; l < 16; l += m < 0 ? 1 : 4) lanes[((o & 3) * 16 + l) * meta + meta - 2 + (o >> 2)] = (uint16_t)slot_off[i];
                    }
        }
        for (int r = 0; r < n_rows; ++r) {
            const int k = row_of[r], m = r / 16, row = r % 16;
            double sum = 0;
            for (int j = c.rowptr[k]; j < c.rowptr[k + 1]; ++j) {
                val[col_slot[c.colidx[j]]] = c.val[j];
                sum += (double)c.val[j] * c.val[j];
            }
            norm = std::max(norm, sum);
            for (int i = 0; i < slots; ++i) {
                const unsigned both = mask[(size_t)r * slots + i];
                if (!both) continue;
                const float *v = &val[(size_t)i * 8];
                for (int nth = 0; nth < kPicks.uses[both]; ++nth) {
                    // (nth uses of a row are nth uses of its tile: the shared ones come first)
                    const int at = where[((size_t)(nth < shared[i] ? 0 : m + 1) * slots + i) * 2 + nth], o = at % 8;
                    uint8_t *rp = &stream[(size_t)(at / 8) * rec];
                    uint16_t *w = reinterpret_cast<uint16_t *>(rp + m * 2048) + ((o / 2) * 16 + row) * 8 + (o % 2) * 4;
                    const Pick &p0 = kPicks.pick[nth][both & 15], &p1 = kPicks.pick[nth][both >> 4];
                    rp[t.mt * 2048 + (((o / 2) * 16 + row) * meta + m) * 2 + o % 2] = (uint8_t)(p0.places | p1.places << 4);
                    auto put = [&](int e, int channel) {
                        const float x = v[channel] * scale;
                        const uint16_t h = x == 0.f ? 0x8000 : to_f16(x);
                        w[e] = h;
                        w[512 + e] = to_f16((x - from_f16(h)) * 2048.f);
                    };
                    for (int e = 0; e < 2; ++e) {
                        if (p0.real[e]) put(e, p0.at[e]);
                        if (p1.real[e]) put(2 + e, 4 + p1.at[e]);
                    }
                }
            }
        }
        return SCONV_OK;
    };
    // (the units are independent; small layers are not worth a thread)
    const int n_all = d.groups * t.n_units;
    std::vector<std::vector<uint8_t>> streams(n_all);
    std::vector<int> status(n_all, SCONV_OK);
    std::vector<double> norm(n_all, 0.0);    // squared, of a unit's largest row
    std::atomic<int> next(0);
    auto work = [&]() {
        for (int u = next++; u < n_all; u = next++) {
            try {
                status[u] = pack_unit(u, streams[u], norm[u]);
            } catch (...) { // (out of a thread it would end the process)
                status[u] = SCONV_ERR_NOMEM;
            }
        }
    };
    std::vector<std::thread> threads;
    try {
        for (int i = 1; c.val.size() > 16384 && i < std::min(n_all, 8); ++i) threads.emplace_back(work);
    } catch (...) { // (no more threads: the ones there are do the work)
    }
    work();
    for (std::thread &th : threads) th.join();
    int64_t n_rec = 0;
    for (int u = 0; u < n_all; ++u) {
        if (status[u]) return status[u];
        for (int b = 0; b < t.nblk; ++b) out.seg[((size_t)u * t.nblk + b) * 2] += (int32_t)n_rec;
        n_rec += (int64_t)(streams[u].size() / rec);
        if (n_rec >= 0x7fffffff / 8) return SCONV_ERR_RANGE;
    }
    out.stream.reserve((size_t)(n_rec + 1) * rec);
    for (const auto &v : streams) out.stream.insert(out.stream.end(), v.begin(), v.end());
    out.stream.resize(out.stream.size() + rec); // the kernel reads one record ahead
    t.stream_bytes = (int64_t)out.stream.size();
    // What is lost of small activations (below 2^-13, see the kernel) takes 2^-36.8 times a row's norm from its sum: 2^-25 of one of
    // 2^-11.8 times the norm.  2^-8, for rows and activations of one sign, whose errors add up.
    t.small_sum = (float)std::ldexp(std::sqrt(*std::max_element(norm.begin(), norm.end())), t.wexp - 8);
    if (t.phased)
        for (int cv = 0; cv < octets * 8; ++cv) {
            const int ph = t.runs ? cv % (s * s) : cv / g.Cg, cl = t.runs ? cv / (s * s) : cv % g.Cg;
            const bool there = cv < t.c_virtual && ph / s < d.R && ph % s < d.S;
            out.choff.push_back(there ? ((cl * d.H + ph / s) * d.W + ph % s) * 4 : SCONV_MFMA_NO_CHANNEL);
        }
    else
        out.choff.push_back(0);
    return SCONV_OK;
}

} // namespace sconv
