// Host checks of the packings that have no inverse in the library: the packed arrays are read the way the kernels read
// them, every address is checked against the buffer the kernel describes, and the sums must be the layer's.  Built by
// test_host_packings.py with the host compiler and linked to libsconv.so; no GPU.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "sconv_internal.h"

using namespace sconv;

static long failures = 0;

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

static const char *name(const sconv_desc &d)
{
    static char s[160];
    std::snprintf(s, sizeof s, "C%d %dx%d K%d %dx%d stride %d pad %d groups %d", d.C, d.H, d.W, d.K, d.R, d.S, d.stride, d.pad, d.groups);
    return s;
}

static float bits(uint64_t e)
{
    const uint32_t u = (uint32_t)e;
    float v;
    std::memcpy(&v, &u, 4);
    return v;
}

// Small integers: every sum below is exact in double and float.
static std::vector<float> ramp(size_t n, int step)
{
    std::vector<float> x(n);
    for (size_t i = 0; i < n; ++i) x[i] = (float)((int)(i * step % 23) - 11);
    return x;
}

static Canonical make_csr(const sconv_desc &d, int keep)
{
    const Geometry g = geometry(d);
    std::vector<float> w((size_t)d.K * g.Cg * d.R * d.S);
    for (size_t i = 0; i < w.size(); ++i) w[i] = (i * 7 + i / 5) % 11 < (size_t)keep ? (float)((int)(i % 13) - 6) : 0.f;
    Canonical c;
    if (build_canonical_from_dense(d, w.data(), c)) std::abort();
    return c;
}

// Output (n, k, y, x) over the zero-padded input.
static double reference(const sconv_desc &d, const Canonical &c, const std::vector<float> &in, int n, int k, int y, int x)
{
    const Geometry g = geometry(d);
    double v = 0;
    for (int j = c.rowptr[k]; j < c.rowptr[k + 1]; ++j) {
        const int col = c.colidx[j], s = col % d.S, r = col / d.S % d.R, ch = k / g.Kg * g.Cg + col / (d.R * d.S);
        const int iy = y * d.stride - d.pad + r, ix = x * d.stride - d.pad + s;
        if (iy >= 0 && iy < d.H && ix >= 0 && ix < d.W) v += (double)c.val[j] * in[(((size_t)n * d.C + ch) * d.H + iy) * d.W + ix];
    }
    return v;
}

// sconv_gather_kernel and sconv_gather4_kernel: a buffer of rec bytes starts shift bytes before the input.  A load the lane
// masks has lane offset 2^31; it reads 0 because that is beyond rec less the scalar offset, which therefore must not be
// negative.  Every other load must lie inside the tensor.
static void check_gather(const sconv_desc &d, int N, int keep)
{
    if (validate_desc(d) != SCONV_OK || !gather_fits(d, N)) return;
    const Geometry g = geometry(d);
    const Canonical c = make_csr(d, keep);
    PackedGather p;
    const int rc = pack_gather(d, c, p);
    CHECK(rc == SCONV_OK, "%s", name(d));
    const std::vector<float> in = ramp((size_t)N * d.C * d.H * d.W, 5);
    const int64_t shift = ((int64_t)d.pad * d.W + d.pad) * 4, bytes = (int64_t)in.size() * 4, rec = bytes + shift;
    const bool four = gather4_fits(d);
    auto load = [&](int64_t at) { // byte offset in the described buffer
        CHECK(at >= shift && at + 4 <= rec && at % 4 == 0, "%s N=%d: byte %ld of %ld", name(d), N, (long)at, (long)rec);
        return at >= shift && at + 4 <= rec ? in[(at - shift) / 4] : 0.f;
    };
    // Bits of the taps that lie inside the image, as the four-position kernel makes them from a position's row and column.
    auto rows_at = [&](int y) {
        uint32_t ones = 0;
        for (int r = 0; r < d.R; ++r) ones |= 1u << r * d.S;
        const int r0 = std::min(std::max(d.pad - y, 0), d.R), r1 = std::min(std::max(d.H + d.pad - y, 0), d.R);
        return ((1u << r1 * d.S) - 1u) & ~((1u << r0 * d.S) - 1u) & ones;
    };
    auto cols_at = [&](int x) {
        const int s0 = std::min(std::max(d.pad - x, 0), d.S), s1 = std::min(std::max(d.W + d.pad - x, 0), d.S);
        return ((1u << s1) - 1u) & ~((1u << s0) - 1u);
    };
    for (int k = 0; k < d.K; ++k) {
        const int j0 = four ? p.rowptr[3 * k] : p.rowptr[k];
        const int n_main = four ? p.rowptr[3 * k + 1] * SCONV_GATHER_CHUNK : p.rowptr[k + 1] - j0, n_edge = four ? p.rowptr[3 * k + 2] : 0;
        CHECK((size_t)j0 + n_main + std::max(n_edge, SCONV_GATHER_CHUNK) <= p.ent.size(), "%s: the chunk read ahead", name(d));
        for (int j = j0; j < j0 + n_main + n_edge; ++j) {
            const int64_t so = (uint32_t)(p.ent[j] >> 32) >> 3 & ~3u;
            CHECK(so <= rec, "%s N=%d: scalar offset %ld beyond the record of %ld bytes", name(d), N, (long)so, (long)rec);
        }
        for (int n = 0; n < N; ++n)
            for (int y = 0; y < g.OH; ++y)
                for (int x = 0; x < g.OW; ++x) {
                    double sum = 0;
                    for (int j = j0; j < j0 + n_main + n_edge; ++j) {
                        const uint32_t ctl = (uint32_t)(p.ent[j] >> 32);
                        const int64_t so = ctl >> 3 & ~3u;
                        const int tap = four ? (int)(ctl & 31) : 31 - (int)(ctl & 31), r = tap / d.S, s = tap % d.S;
                        const int iy = y * d.stride - d.pad + r, ix = x * d.stride - d.pad + s;
                        const bool seen = tap < d.R * d.S && iy >= 0 && iy < d.H && ix >= 0 && ix < d.W;
                        const int64_t base = ((int64_t)n * d.C * d.H * d.W + (y * d.W + x) * d.stride) * 4;
                        if (four && j < j0 + n_main) { // the four words are loaded whatever the mask says
                            for (int i = 0; x % 4 == 0 && i < 4; ++i) (void)load(base + so + 4 * i);
                        }
                        if (seen) sum += (double)bits(p.ent[j]) * load(base + so);
                    }
                    if (four)
                        for (int tap = 0; tap < d.R * d.S; ++tap) {
                            const int iy = y - d.pad + tap / d.S, ix = x - d.pad + tap % d.S;
                            CHECK((cols_at(x) * rows_at(y) >> tap & 1) == (iy >= 0 && iy < d.H && ix >= 0 && ix < d.W), "%s: tap %d at %d %d", name(d), tap, y, x);
                        }
                    const double want = reference(d, c, in, n, k, y, x);
                    CHECK(sum == want, "%s N=%d output %d %d %d %d: %g instead of %g", name(d), N, n, k, y, x, sum, want);
                }
        // fours of positions counted through the image: they pass the end of a row, and of the image
        if (!four || g.OW != d.W || g.OW < 4) continue;
        for (int n = 0; n < N; ++n)
            for (int x0 = 0; x0 < g.OH * g.OW; x0 += 4) {
                const int y = x0 / g.OW, x = x0 - y * g.OW;
                uint32_t valid[4];
                for (int i = 0; i < 4; ++i) {
                    const bool over = x + i >= g.OW;
                    valid[i] = x0 + i < g.OH * g.OW ? cols_at(over ? x + i - g.OW : x + i) * rows_at(over ? y + 1 : y) : 0;
                }
                double sum[4] = {};
                for (int j = j0; j < j0 + n_main + n_edge; ++j) {
                    const uint32_t ctl = (uint32_t)(p.ent[j] >> 32);
                    const int64_t base = ((int64_t)n * d.C * d.H * d.W + x0) * 4, so = ctl >> 3 & ~3u;
                    for (int i = 0; i < 4; ++i) {
                        const bool seen = valid[i] >> (ctl & 31) & 1;
                        const float v = j < j0 + n_main || seen ? load(base + so + 4 * i) : 0.f;
                        if (seen) sum[i] += (double)bits(p.ent[j]) * v;
                    }
                }
                for (int i = 0; i < 4 && x0 + i < g.OH * g.OW; ++i) {
                    const double want = reference(d, c, in, n, k, (x0 + i) / g.OW, (x0 + i) % g.OW);
                    CHECK(sum[i] == want, "%s N=%d output %d %d at %d: %g instead of %g", name(d), N, n, k, x0 + i, sum[i], want);
                }
            }
    }
}

static void gather_cases()
{
    const int sizes[] = {1, 2, 3, 5}, taps[] = {1, 2, 3, 5};
    for (int H : sizes)
        for (int W : sizes)
            for (int R : taps)
                for (int S : taps)
                    for (int pad = 0; pad <= 3; ++pad)
                        for (int stride = 1; stride <= 3; ++stride)
                            for (int C = 1; C <= 4; ++C)
                                for (int groups = 1; groups <= (C % 2 == 0 ? 2 : 1); ++groups)
                                    for (int N = 1; N <= 2; ++N) check_gather({C, H, W, 2, R, S, stride, pad, groups}, N, (H + S) % 2 ? 11 : 5);
    check_gather({512, 1, 1, 3, 3, 3, 1, 1, 1}, 1, 11);
    check_gather({64, 7, 6, 5, 3, 3, 1, 1, 2}, 3, 4);
    for (int W : {4, 5, 6, 7, 9, 13})
        for (int R : {1, 2, 3, 5})
            for (int S : {1, 3, 5, 7}) check_gather({4, 6, W, 2, R, S, 1, S / 2, W % 2 ? 1 : 2}, 2, W % 3 ? 11 : 6);
    check_gather({6, 9, 7, 4, 31, 1, 1, 15, 1}, 1, 11);
    check_gather({6, 1, 2, 4, 31, 1, 2, 15, 1}, 1, 11);
    check_gather({5, 2, 1, 4, 1, 31, 1, 15, 1}, 1, 11);
}

static void fc_gather_cases()
{
    for (int C : {1, 3, 64, 333})
        for (int keep : {0, 2, 11}) {
            const sconv_desc d = {C, 1, 1, 5, 1, 1, 1, 0, 1};
            const Canonical c = make_csr(d, keep);
            PackedGather p;
            CHECK(pack_fc_gather(d, c, p) == SCONV_OK, "%s", name(d));
            CHECK(p.rowptr == c.rowptr && p.ent.size() == c.val.size(), "%s", name(d));
            for (size_t j = 0; j < p.ent.size(); ++j)
                CHECK(bits(p.ent[j]) == c.val[j] && (int)(p.ent[j] >> 32) == c.colidx[j] && c.colidx[j] < C, "%s entry %zu", name(d), j);
        }
}

// sconv_mfma_kernel: fragments read back to (filter, column) through the depth octets' offsets and the channel table, the
// three parts added up.  Every weight once (a stored zero as -0), zeros everywhere else, offsets inside the staged block.
static void check_mfma_packing(const sconv_desc &layer, const MfmaTiling &t, int keep, bool small_weights)
{
    const sconv_desc d = mfma_desc(layer);
    const Geometry g = geometry(d);
    Canonical c = make_csr(layer, keep);
    for (size_t j = 0; j < c.val.size(); ++j) // all 24 bits, over the whole range the kernel takes
        c.val[j] = std::ldexp(1.0f + (float)(j * 2654435761u % (1u << 23)) / (1 << 23), small_weights ? (int)(j % 210) - 94 : 0) * (j % 2 ? -1.f : 1.f);
    for (size_t j = 5; j < c.val.size(); j += 17) c.val[j] = j % 2 ? -0.f : 0.f;
    PackedMfma p;
    CHECK(pack_mfma(layer, c, t, p) == SCONV_OK, "%s", name(layer));
    const int s = t.phased ? d.stride : 1, cols = g.Cg * d.R * d.S, octets = (t.c_virtual + 7) / 8, g8_last = octets - (t.nblk - 1) * t.g8;
    CHECK(t.c_virtual == g.Cg * s * s && g8_last >= 1 && g8_last <= t.g8, "%s", name(layer));
    CHECK((int)p.uoff.size() == 2 * (t.steps + t.steps_last), "%s", name(layer));
    for (int u : p.uoff) CHECK(u >= 0 && u % 48 == 0 && u < t.g8 * t.plane * 48, "%s: depth octet at %d", name(layer), u);
    if (t.phased)
        for (int cv = 0; cv < octets * 8; ++cv) {
            const int off = p.choff[cv], ph = cv / g.Cg;
            if (off < 0) { // bit 31 masks the lane; the rest is the scalar offset, which the range check uses
                CHECK((off & 0x7fffffff) == 0, "%s: missing channel %d has offset %d", name(layer), cv, off);
                CHECK(cv >= t.c_virtual || ph / s >= d.R || ph % s >= d.S, "%s: channel %d is missing", name(layer), cv);
                continue;
            }
            CHECK(cv < t.c_virtual && off < g.Cg * d.H * d.W * 4, "%s: channel %d at %d", name(layer), cv, off);
            CHECK(off == ((cv % g.Cg * d.H + ph / s) * d.W + ph % s) * 4, "%s: channel %d", name(layer), cv);
        }
    const size_t tile = (size_t)t.total_steps * 1536;
    CHECK(p.wfrag.size() == (size_t)d.groups * t.n_tiles32 * tile + 1536, "%s", name(layer));
    std::vector<float> got((size_t)d.K * cols, 0.f);
    std::vector<char> there(got.size(), 0);
    for (int grp = 0; grp < d.groups; ++grp)
        for (int t32 = 0; t32 < t.n_tiles32; ++t32)
            for (int step = 0; step < t.total_steps; ++step) {
                const int b = std::min(step / t.steps, t.nblk - 1), last = b == t.nblk - 1;
                for (int lane = 0; lane < 64; ++lane)
                    for (int e = 0; e < 8; ++e) {
                        const uint16_t *at = &p.wfrag[((size_t)(grp * t.n_tiles32 + t32) * t.total_steps + step) * 1536 + lane * 8 + e];
                        float part[3];
                        for (int i = 0; i < 3; ++i) {
                            const uint32_t u = (uint32_t)at[i * 512] << 16;
                            std::memcpy(&part[i], &u, 4);
                        }
                        const float v = part[0] + (part[1] + part[2]);
                        if (v == 0.f && at[0] == 0 && at[512] == 0 && at[1024] == 0) continue;
                        const int u = 2 * (step - b * t.steps) + lane / 32, kl = t32 * 32 + lane % 32;
                        const int cell = p.uoff[(last ? 2 * t.steps : 0) + u] / 48, cv = (b * t.g8 + cell / t.plane) * 8 + e;
                        const int fr = cell % t.plane / t.Wl, fs = cell % t.plane % t.Wl, ph = cv / g.Cg;
                        const int r = fr * s + (t.phased ? ph / s : 0), col_s = fs * s + (t.phased ? ph % s : 0), ch = t.phased ? cv % g.Cg : cv;
                        const bool ok = kl < g.Kg && cv < t.c_virtual && r < d.R && col_s < d.S;
                        CHECK(ok, "%s: a weight at row %d channel %d tap %d %d", name(layer), kl, cv, r, col_s);
                        if (!ok) continue;
                        const size_t to = (size_t)(grp * g.Kg + kl) * cols + (ch * d.R + r) * d.S + col_s;
                        CHECK(!there[to] && (v != 0.f || (at[0] == 0x8000 && at[512] == 0 && at[1024] == 0)), "%s: weight %zu", name(layer), to);
                        got[to] = v * SCONV_MFMA_SCALE;
                        there[to] = 1;
                    }
            }
    for (int k = 0; k < d.K; ++k)
        for (int j = c.rowptr[k]; j < c.rowptr[k + 1]; ++j) {
            const size_t at = (size_t)k * cols + c.colidx[j];
            CHECK(there[at] && got[at] == c.val[j], "%s: weight %d %d is %g instead of %g", name(layer), k, c.colidx[j], got[at], c.val[j]);
            there[at] = 0;
        }
    for (char t : there) CHECK(!t, "%s: a weight that is not stored", name(layer));
}

// The column kernel's tiling: blocks of whole steps that depend on the layer alone, no part without blocks, a block in LDS.
static bool check_column(const sconv_desc &layer, int N, const MfmaTiling &staged, int min_splits, MfmaTiling &t)
{
    t = staged;
    const bool ok = choose_mfma_column(layer, N, min_splits, t);
    CHECK(ok, "%s N=%d: no tiling of %d parts or more", name(layer), N, min_splits);
    if (!ok) return false;
    const int octets = (t.c_virtual + 7) / 8, g8_last = octets - (t.nblk - 1) * t.g8, blk_split = (t.nblk + t.splits - 1) / t.splits;
    CHECK(t.column && t.nt == 1 && (t.mt == 1 || t.mt == 2) && t.mt <= t.n_tiles32 && t.us > 0, "%s", name(layer));
    CHECK(t.g8 >= 1 && t.g8 <= 16 && (t.nblk == 1 || t.g8 % 2 == 0) && g8_last >= 1 && g8_last <= t.g8, "%s: %d blocks of %d octets", name(layer), t.nblk, t.g8);
    CHECK(t.steps == (t.g8 + 1) / 2 && t.steps_last == (g8_last + 1) / 2 && t.total_steps == (t.nblk - 1) * t.steps + t.steps_last, "%s: steps", name(layer));
    CHECK(t.total_steps == (t.c_virtual + 15) / 16, "%s: steps of 16 channels", name(layer));
    CHECK(t.splits >= min_splits && (t.splits - 1) * blk_split < t.nblk, "%s N=%d: %d parts of %d blocks", name(layer), N, t.splits, t.nblk);
    CHECK(t.lds_bytes >= t.g8 * t.plane * 48 + 8 * (t.steps + t.steps_last) + 4 * t.plane && t.lds_bytes <= 80 * 1024, "%s: %d bytes of LDS", name(layer), t.lds_bytes);
    return true;
}

static void check_mfma(const sconv_desc &layer, int N, int keep, bool small_weights)
{
    MfmaTiling t, column, other;
    if (validate_desc(layer) != SCONV_OK || !choose_mfma(layer, N, t)) return;
    check_mfma_packing(layer, t, keep, small_weights);
    if (!t.one_tap || !check_column(layer, N, t, 1, column)) return;
    check_mfma_packing(layer, column, keep, small_weights);
    if (choose_mfma(layer, 4 * N, t) && check_column(layer, 4 * N, t, t.splits, other))
        CHECK(other.g8 == column.g8 && other.nblk == column.nblk, "%s: another packing for another batch size", name(layer));
}

// Every number of channels finds a column tiling with the parts that the staged kernel would make.
static void column_cases()
{
    for (int C = 1; C <= 2600; C += C < 600 ? 1 : 7)
        for (int K : {24, 200})
            for (int N : {1, 8, 64, 1000}) {
                const sconv_desc conv = {C, 7, 7, K, 1, 1, 1, 0, 1}, fc = {C, 1, 1, K, 1, 1, 1, 0, 1};
                for (const sconv_desc &d : {conv, fc}) {
                    MfmaTiling t, column;
                    if (!choose_mfma(d, N, t)) continue;
                    CHECK(t.one_tap, "%s", name(d));
                    check_column(d, N, t, 1, column);
                    check_column(d, N, t, t.splits, column);
                }
            }
}

static void mfma_cases()
{
    for (int C : {1, 3, 8, 13, 40})
        for (int K : {1, 33, 70})
            for (int R : {1, 3, 4})
                for (int S : {1, 2, 5})
                    for (int stride = 1; stride <= 3; ++stride)
                        for (int pad = 0; pad <= 1; ++pad)
                            for (int groups = 1; groups <= 2; ++groups)
                                check_mfma({C * groups, 9, 11, K * groups, R, S, stride, pad, groups}, 3, 6, R == S || stride == 2);
    for (int stride = 2; stride <= 5; ++stride)
        for (int H = 2; H <= 4; ++H) check_mfma({3, H, 2, 40, 2, 1, stride, 0, 1}, 3, 11, false);
    check_mfma({3, 67, 67, 96, 11, 11, 4, 0, 1}, 24, 11, false);
    check_mfma({301, 16, 16, 40, 3, 3, 2, 1, 1}, 7, 11, true);
    check_mfma({200, 14, 14, 70, 1, 1, 1, 0, 1}, 60, 4, true);
    check_mfma({777, 1, 1, 100, 1, 1, 1, 0, 1}, 1024, 9, true);
    for (int C : {15, 17, 41, 96, 100, 101, 202, 250, 777}) check_mfma({2 * C, 9, 11, 66, 1, 1, 1, 0, 2}, 12, 9, C % 2 == 1);
    column_cases();
}

int main(int argc, char **argv)
{
    const char *what = argc > 1 ? argv[1] : "";
    if (!std::strcmp(what, "gather"))
        gather_cases();
    else if (!std::strcmp(what, "fc_gather"))
        fc_gather_cases();
    else if (!std::strcmp(what, "mfma"))
        mfma_cases();
    else
        return 2;
    std::printf("%ld failures\n", failures);
    return failures ? 1 : 0;
}
