// Host check of the flat streams packed for the matrix cores: records decoded the way sconv_flat_mc_kernel feeds them to
// v_smfmac_f32_16x16x64_f16, every weight of the layer found once and within the split's precision, every LDS address inside
// the staged block; the streams walked by the kernel's own lines, every step on its record.  Built by test_host_flat_mc.py and linked to libsconv.so; no GPU.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "sconv_internal.h"
#include "sconv_mc_walk.h"

using namespace sconv;

static long failures = 0, layers = 0, private_steps = 0, twice = 0, empty_blocks = 0;

#define CHECK(cond, ...) \
    do { \
        if (!(cond)) { \
            if (++failures <= 20) { \
                std::printf("FAIL %s: ", #cond); \
                std::printf(__VA_ARGS__); \
                std::printf("\n"); \
            } \
        } \
    } while (0)

static uint32_t seed = 7;
static double uniform() { return (double)((seed = seed * 1664525u + 1013904223u) >> 8) / (1 << 24); }

static double f16(uint16_t b)
{
    const int e = b >> 10 & 31, m = b & 1023;
    const double v = e == 0 ? std::ldexp(m, -24) : std::ldexp(m + 1024, e - 25);
    return b & 0x8000 ? -v : v;
}

// A wave's way through its part of the stream, for every way to split the channel blocks over workgroups.
static void walk(const PackedFlatMc &p, const FlatMcTiling &t, int units, const char *what)
{
    const int rec = SCONV_MC_RECORD(t.mt);
    struct Record {
        int at = -1;         // in the stream, -1 where nothing was loaded
        int off = -1;        // the record that its LDS addresses are from
    };
    for (int u = 0; u < units; ++u)
        for (int splits = 1; splits <= t.nblk; ++splits) {
            const int per = (t.nblk + splits - 1) / splits;
            const int32_t *seg = &p.seg[(size_t)u * t.nblk * 2];
            for (int b_first = 0; b_first < t.nblk; b_first += per) {
                int64_t pos = 0;
                int since = 0, added = 0, done = 0;   // steps that the totals had when they were last added to, all steps
                Record r0;
                auto load = [&](Record &r) {
                    r.at = r.off = seg[2 * b_first] + (int)(pos / rec);
                    pos += rec;
                    CHECK((int64_t)(r.at + 1) * rec <= t.stream_bytes, "a record past the end: %s", what);
                };
                for (int b = b_first; b < std::min(b_first + per, t.nblk); ++b) {
                    const int n_shared = seg[2 * b + 1] & 0xffff, n_private = seg[2 * b + 1] >> 16;
                    int steps = 0;
                    bool own = false;
                    pos = mc_block_at(seg, b, b_first, rec);
                    load(r0);
                    auto step = [&](const Record &cur, const Record &next) {
                        CHECK(cur.off >= 0 && next.off >= 0, "unit %d block %d step %d of %d: LDS read at an address that no record gave: %s", u, b,
                              steps, n_shared + n_private, what);
                        CHECK(cur.at == seg[2 * b] + steps, "unit %d block %d step %d on record %d: %s", u, b, steps, cur.at - seg[2 * b], what);
                        CHECK(own == (steps >= n_shared), "%s", what);
                        ++steps;
                        own = steps >= n_shared;
                    };
                    own = n_shared == 0;
                    mc_walk_block(r0, n_shared, n_private, since, load, step, step, [&](int left) {
                        CHECK(left == n_shared + n_private - steps, "%s", what);
                        CHECK(done + steps - added <= 7, "%d steps in the accumulators: %s", done + steps - added, what);
                        added = done + steps;
                    });
                    done += steps;
                    CHECK(done - added <= 6, "%d steps in the accumulators after block %d: %s", done - added, b, what);
                    CHECK(steps == n_shared + n_private, "%s", what);
                    empty_blocks += splits == 1 && steps == 0 && b + 1 < t.nblk;
                }
            }
        }
}

// no_first .. no_last: input channels of a group that no filter has weights on; short_row: a filter of 16 nonzeros in one channel
static void check(const sconv_desc &layer, int N, double density, bool skewed, bool explicit_zeros, int no_first = 0, int no_last = -1,
                  bool short_row = false)
{
    const Geometry lg = geometry(layer);
    const int cols = lg.Cg * layer.R * layer.S;
    std::vector<int32_t> rowptr(1, 0), col;
    std::vector<float> val;
    for (int k = 0; k < layer.K; ++k) {
        const double dk = skewed ? (k % 5 == 0 ? 0.0 : density * (0.3 + 1.7 * uniform())) : density;
        for (int j = 0; j < cols; ++j)
            if (short_row && k == layer.K - 1 ? j >= cols / 2 && j < cols / 2 + 16
                                              : uniform() < dk && !(j / (layer.R * layer.S) >= no_first && j / (layer.R * layer.S) <= no_last)) {
                col.push_back(j);
                val.push_back(explicit_zeros && j % 7 == 0 ? 0.f : (float)((uniform() + 0.001) * (uniform() < 0.5 ? -1 : 1)));
            }
        rowptr.push_back((int32_t)col.size());
    }
    Canonical c;
    if (build_canonical_from_arrays(layer, rowptr.data(), col.data(), val.data(), c)) std::abort();
    FlatMcTiling t;
    if (!mfma_fits(layer, N, false) || !choose_flat_mc(layer, c, N, N % 2 == 0, t)) return;
    const sconv_desc d = mfma_desc(layer);
    const Geometry g = geometry(d);
    PackedFlatMc p;
    char what[200];
    std::snprintf(what, sizeof what, "C%d %dx%d K%d %dx%d stride %d pad %d groups %d N=%d density %g: mt %d nt %d wr %d g8 %d plane %d", layer.C, layer.H,
                  layer.W, layer.K, layer.R, layer.S, layer.stride, layer.pad, layer.groups, N, density, t.mt, t.nt, t.wr, t.g8, t.plane);
    if (pack_flat_mc(d, c, t, p) != SCONV_OK) {
        CHECK(false, "not packed: %s", what);
        return;
    }
    ++layers;
    const int rec = SCONV_MC_RECORD(t.mt), octets = (t.c_virtual + 7) / 8, s = t.phased ? d.stride : 1, rows = 16 * t.mt, meta = (t.mt + 1) / 2 * 2 + 2;
    CHECK((int64_t)p.stream.size() == t.stream_bytes && p.stream.size() % rec == 0, "%s", what);
    CHECK(p.seg.size() == (size_t)d.groups * t.n_units * t.nblk * 2 && p.row_of.size() == (size_t)d.groups * t.n_units * rows, "%s", what);
    CHECK(t.n_units * rows >= g.Kg && t.n_units % t.wr == 0, "%s", what);
    CHECK((int64_t)t.g8 * t.octet * 16 + 8 * t.plane + 16 <= t.lds_bytes && t.lds_bytes % 16 == 0 && t.lds_bytes <= 80 * 1024, "%s", what);
    CHECK(4 * SCONV_MC_STORE_BYTES(t.mt, t.nt) + 16 <= t.lds_bytes, "%s", what);
    CHECK((t.nblk - 1) * t.g8 < octets && t.nblk * t.g8 >= octets, "%s", what);
    std::vector<double> got((size_t)d.K * cols, 0.0);
    std::vector<int> seen((size_t)d.K * cols, 0), rows_seen(d.K, 0);
    int64_t next = 0;
    for (int u = 0; u < d.groups * t.n_units; ++u) {
        const int grp = u / t.n_units;
        for (int r = 0; r < rows; ++r) {
            const int k = p.row_of[(size_t)u * rows + r];
            if (k < 0) continue;
            CHECK(k / g.Kg == grp, "row %d in group %d: %s", k, grp, what);
            ++rows_seen[k];
        }
        for (int b = 0; b < t.nblk; ++b) {
            const int o8 = std::min(t.g8, octets - b * t.g8);
            const int32_t *seg = &p.seg[((size_t)u * t.nblk + b) * 2];
            const int n_shared = seg[1] & 0xffff, n_private = seg[1] >> 16;
            CHECK(seg[0] == next, "records follow each other: %s", what);
            next += n_shared + n_private;
            private_steps += n_private;
            for (int i = 0; i < n_shared + n_private; ++i) {
                const uint8_t *r = &p.stream[(size_t)(seg[0] + i) * rec];
                for (int m = 0; m < t.mt; ++m) {
                    const uint16_t *h = reinterpret_cast<const uint16_t *>(r + m * 2048), *l = h + 512;
                    const uint16_t *places = reinterpret_cast<const uint16_t *>(r + t.mt * 2048);
                    for (int o = 0; o < 8; ++o) {
                        int at = -1;
                        for (int z = 0; z < 16; ++z) {
                            const int word = places[((o & 3) * 16 + z) * meta + meta - 2 + (o >> 2)];
                            if (i < n_shared) CHECK(at < 0 || at == word, "one address for the quarter: %s", what);
                            if (i < n_shared || (z & 3) == m) at = word;
                        }
                        const int ol = at / t.octet, cell = at % t.octet, tr = cell / t.pitch, ts = cell % t.pitch;
                        CHECK(ol < o8 && tr < t.Rr && ts < t.Sr, "octet %d, tap %d %d: %s", ol, tr, ts, what);
                        for (int row = 0; row < 16; ++row) {
                            const int lane = (o / 2) * 16 + row, idx = places[lane * meta + m] >> (8 * (o % 2)) & 255;
                            for (int e = 0; e < 4; ++e) {
                                const size_t w = (size_t)lane * 8 + (o % 2) * 4 + e;
                                const int place = idx >> (2 * e) & 3;
                                if (e % 2) CHECK(place > (idx >> (2 * e - 2) & 3), "places in order: %s", what);
                                if (h[w] == 0) { // not a stored weight
                                    CHECK(l[w] == 0, "%s", what);
                                    continue;
                                }
                                const int k = p.row_of[(size_t)u * rows + m * 16 + row], cv = (b * t.g8 + ol) * 8 + (e / 2) * 4 + place;
                                const int ph = !t.phased ? 0 : t.runs ? cv % (s * s) : cv / g.Cg, cl = !t.phased ? cv : t.runs ? cv / (s * s) : cv % g.Cg;
                                const int fr = tr * s + ph / s, fs = ts * s + ph % s;
                                if (k < 0 || cv >= t.c_virtual || fr >= d.R || fs >= d.S) {
                                    CHECK(false, "a weight that the layer does not have: %s", what);
                                    continue;
                                }
                                const size_t where = (size_t)k * cols + (cl * d.R + fr) * d.S + fs;
                                got[where] = std::ldexp(f16(h[w]) + f16(l[w]) / 2048, -t.wexp);
                                ++seen[where];
                            }
                        }
                    }
                }
            }
        }
    }
    CHECK((size_t)(next + 1) * rec == p.stream.size(), "a spare record: %s", what);
    for (int k = 0; k < d.K; ++k) {
        CHECK(rows_seen[k] == 1, "row %d: %s", k, what);
        int j = c.rowptr[k];
        for (int i = 0; i < cols; ++i) {
            const bool there = j < c.rowptr[k + 1] && c.colidx[j] == i;
            const double want = there ? c.val[j] : 0.0;
            j += there;
            CHECK(seen[(size_t)k * cols + i] == (there ? 1 : 0), "row %d column %d packed %d times: %s", k, i, seen[(size_t)k * cols + i], what);
            CHECK(std::fabs(got[(size_t)k * cols + i] - want) <= std::fabs(want) * 0x1p-23, "row %d column %d: %s", k, i, what);
        }
    }
    for (size_t i = 0; i < p.seg.size(); i += 2) twice += p.seg[i + 1] & 0xffff;
    walk(p, t, d.groups * t.n_units, what);
    // Staged as the kernel stages (cell numbers for values), then every position reads every tap: the input element or the zero
    // of the padding, from both parts.
    const int pos_waves = t.wr == 2 ? 2 : 4, bn = 16 * t.nt * pos_waves, OHW = g.OH * g.OW, row_img = (g.OH - 1) * t.lstep + t.Rr;
    const int64_t P = (int64_t)N * OHW;
    for (int64_t p0 = 0; p0 < P; p0 += bn) {
        const int n0 = (int)(p0 / OHW), y0 = (int)(p0 % OHW) / g.OW, rows_first = (g.OH - 1 - y0) * t.lstep + t.Rr;
        auto row_at = [&](int n, int y) { return n == n0 ? (y - y0) * t.lstep : rows_first + (n - n0 - 1) * row_img + y * t.lstep; };
        const int64_t p1 = std::min(p0 + bn, P) - 1;
        const int cells = (row_at((int)(p1 / OHW), (int)(p1 % OHW) / g.OW) + t.Rr) * t.Wl;
        CHECK(cells <= t.plane && (cells + 63) / 64 <= 16, "cells %d: %s", cells, what);
        std::vector<int64_t> block((size_t)t.g8 * t.octet, 0);
        for (int ol : {0, t.g8 - 1})
            for (int cell = 0; cell < cells; ++cell) {
                const int row = cell / t.Wl, col = cell % t.Wl;
                int n = 0, yp = y0 * t.lstep + row;
                if (row >= rows_first) {
                    n = 1 + (row - rows_first) / row_img;
                    yp = (row - rows_first) % row_img;
                }
                const int iy = yp * t.cstep - d.pad, ix = col * t.cstep - d.pad;
                const bool ok = iy >= 0 && iy < d.H && ix >= 0 && ix < d.W;
                const size_t at = (size_t)ol * t.octet + row * t.pitch + col;
                CHECK(at + t.part < block.size() && (t.part >= t.octet / 2 || col < t.part), "%s", what);
                block[at] = ok ? 1 + 2 * ((((int64_t)n0 + n) * d.H + iy) * d.W + ix) : 0;
                block[at + t.part] = ok ? 2 + 2 * ((((int64_t)n0 + n) * d.H + iy) * d.W + ix) : 0;
            }
        for (int64_t q = p0; q <= p1; ++q) {
            const int n = (int)(q / OHW), y = (int)(q % OHW) / g.OW, x = (int)(q % g.OW);
            for (int ol : {0, t.g8 - 1})
                for (int tr = 0; tr < t.Rr; ++tr)
                    for (int ts = 0; ts < t.Sr; ++ts) {
                        const size_t at = (size_t)ol * t.octet + (row_at(n, y) + tr) * t.pitch + x * t.lstep + ts;
                        // (phase form: the phase's offset is the channel's, the taps that no weight has may leave the image)
                        const int iy = (y * t.lstep + tr) * t.cstep - d.pad, ix = (x * t.lstep + ts) * t.cstep - d.pad;
                        const bool ok = iy >= 0 && iy < d.H && ix >= 0 && ix < d.W;
                        const int64_t want = ok ? 1 + 2 * (((int64_t)n * d.H + iy) * d.W + ix) : 0;
                        CHECK(at + t.part < block.size(), "%s", what);
                        CHECK(block[at] == want && block[at + t.part] == (ok ? want + 1 : 0), "position %ld tap %d %d: %s", (long)q, tr, ts, what);
                    }
        }
    }
}

int main()
{
    const int strides[] = {1, 1, 1, 2, 3};
    for (int i = 0; i < 420; ++i) {
        const int groups = uniform() < 0.3 ? 2 : 1, r = 1 + (int)(uniform() * 5) % 5, stride = strides[(int)(uniform() * 5)];
        const int hw = 4 + (int)(uniform() * 34);
        sconv_desc d = {groups * (8 + (int)(uniform() * 90)), hw, 3 + (int)(uniform() * 36), groups * (1 + (int)(uniform() * 160)), r,
                        uniform() < 0.8 ? r : 1 + (int)(uniform() * 4), stride, (int)(uniform() * (r / 2 + 1)), groups};
        if (validate_desc(d) != SCONV_OK) continue;
        check(d, 1 + (int)(uniform() * 9), i % 7 == 0 ? 1.0 : 0.06 + 0.6 * uniform(), i % 3 == 0, i % 4 == 0);
    }
    check({96, 27, 27, 256, 5, 5, 1, 2, 2}, 3, 0.1, false, false);
    check({3, 227, 227, 96, 11, 11, 4, 0, 1}, 1, 0.3, false, false);
    check({600, 1, 1, 300, 1, 1, 1, 0, 1}, 64, 0.2, false, false);
    check({384, 13, 13, 192, 3, 3, 1, 1, 1}, 2, 0.1, true, false);
    // channels that pruning took from every filter: first, middle and last blocks of the stream without records
    for (int lo : {0, 32, 96})
        for (int groups : {1, 2})
            for (int hi : {lo + 31, lo + 40, lo + 90}) {
                check({128 * groups, 28, 28, 96 * groups, 3, 3, 1, 1, groups}, 3, 0.3, false, false, lo, std::min(hi, 127));
                check({128 * groups, 14, 14, 40 * groups, 3, 3, 1, 1, groups}, 2, 0.8, false, false, lo, std::min(hi, 127));
                check({128 * groups, 28, 28, 40 * groups, 3, 3, 2, 0, groups}, 3, 0.4, false, false, lo, std::min(hi, 127));
            }
    check({256, 13, 13, 384, 3, 3, 1, 1, 1}, 256, 0.2, false, false, 0, 95);
    check({256, 13, 13, 384, 3, 3, 1, 1, 1}, 256, 0.2, false, false, 88, 175);
    check({128, 28, 28, 65, 3, 3, 1, 1, 1}, 3, 0.3, false, false, 0, -1, true);   // a wave of one short row
    check({40, 40, 40, 64, 3, 3, 4, 0, 1}, 3, 0.7, false, false);                 // phases that no tap of the filter has
    CHECK(layers > 200 && private_steps > 100 && twice > 1000 && empty_blocks > 50, "%ld layers, %ld private steps, %ld empty blocks", layers,
          private_steps, empty_blocks);
    std::printf("%ld layers, %ld private steps of %ld, %ld empty blocks before others, %ld failures\n", layers, private_steps, twice, empty_blocks,
                failures);
    return failures ? 1 : 0;
}
