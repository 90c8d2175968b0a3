// Host checks of which kernel a call goes to.  The device side of libsconv (launches, uploads, events) is replaced by the
// functions below: this program defines the same symbols, and the library's calls resolve to them.  Built and linked to
// libsconv.so by test_host_dispatch.py; no GPU.
#include <dlfcn.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "sconv_internal.h"

using namespace sconv;

static std::string launched;              // the kernels of the last call, in order
static int uploads_ok, uploads_fail;      // the next uploads that succeed, then those that fail; all others succeed
static size_t uploaded;                   // bytes of all uploads
static std::map<std::string, float> cost; // what a launch of a kernel is to take, in ms (1 unless given)
static float clock_ms;

static int packs; // flat-stream packings made

namespace sconv {
int pack_flat(const sconv_desc &d, const Canonical &c, const LdsTiling &t, PackedFlat &out)
{
    using F = int (*)(const sconv_desc &, const Canonical &, const LdsTiling &, PackedFlat &);
    static const F real = (F)dlsym(RTLD_NEXT, "_ZN5sconv9pack_flatERK10sconv_descRKNS_9CanonicalERKNS_9LdsTilingERNS_10PackedFlatE");
    if (!real) std::abort();
    ++packs;
    return real(d, c, t, out);
}
static int ran(const char *what)
{
    launched += launched.empty() ? what : std::string("+") + what;
    const auto c = cost.find(what);
    clock_ms += c == cost.end() ? 1.f : c->second;
    return SCONV_OK;
}
int launch_lds(const sconv_desc &, const LdsTiling &, const DeviceLds &, const float *, float *, int, void *, int *) { return ran("rows"); }
int launch_lds2(const sconv_desc &, const LdsTiling &, const DeviceLds &dev, const Lds2Layout &, const float *, float *, int, const Epilogue &,
                int64_t, void *, int *)
{
    if (!dev.pairs || !dev.store_tbl) std::abort();
    return ran("flat");
}
int launch_direct(const sconv_desc &, const DeviceDirect &, const float *, float *, int, void *, int *) { return ran("direct"); }
int launch_phase(const sconv_desc &, const sconv_desc &, const float *, float *, int, void *, int *) { return ran("phase"); }
int launch_reduce(const float *, float *, int, int64_t, int64_t, int, const Epilogue &, void *, int *) { return ran("reduce"); }
int launch_epilogue(float *, int64_t, int64_t, int, const Epilogue &ep, void *, int *) { return ep.bias || ep.relu ? ran("epilogue") : SCONV_OK; }
int launch_gather(const sconv_desc &, const DeviceGather &dev, const GatherShape &, const float *, float *, int, const Epilogue &, void *, int *)
{
    if (!dev.ent) std::abort();
    return ran("gather");
}
int launch_fc_gather(const sconv_desc &, const DeviceGather &dev, const GatherShape &, const float *, float *, int, const Epilogue &, void *, int *)
{
    if (!dev.ent) std::abort();
    return ran("fc_gather");
}
static bool column; // the last launch on the matrix cores was the column kernel's
int launch_mfma(const sconv_desc &, const MfmaTiling &t, const DeviceMfma &dev, const DeviceDirect &direct, const float *, float *, int, bool,
                const Epilogue &, int64_t, void *, int *)
{
    if (!dev.wfrag || (dev.short_rows && !direct.trip)) std::abort();
    column = t.column;
    return ran("mfma");
}
int launch_flat_mc(const sconv_desc &, const FlatMcTiling &t, const DeviceLds &dev, const float *, float *, int, const Epilogue &, int64_t, void *, int *)
{
    if (!dev.pairs || !dev.seg_ptr || !dev.row_of || !dev.store_tbl || t.stream_bytes < 1 || t.nt < 2) std::abort();
    return ran("flat_mc");
}
int upload(const void *, size_t bytes, void **dev, int *hip_err)
{
    *dev = nullptr;
    if (uploads_ok > 0) {
        --uploads_ok;
    } else if (uploads_fail > 0) {
        --uploads_fail;
        *hip_err = 2;
        return SCONV_ERR_HIP;
    }
    *dev = std::malloc(1); // (never read; freed by release)
    uploaded += bytes;
    return SCONV_OK;
}
void release(void *dev) { std::free(dev); }
int static_scratch(void **base, size_t *bytes, int *)
{
    *base = (void *)(size_t)4096;
    *bytes = SCONV_NOALLOC_SCRATCH_BYTES;
    return SCONV_OK;
}
static float started;
int timer_create(StreamTimer &, int *) { return SCONV_OK; }
int timer_start(StreamTimer &, void *, int *)
{
    started = clock_ms;
    return SCONV_OK;
}
int timer_stop_ms(StreamTimer &, void *, float *ms, int *)
{
    *ms = clock_ms - started;
    return SCONV_OK;
}
void timer_destroy(StreamTimer &) {}
} // namespace sconv

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

static float *const in = (float *)(size_t)65536, *const out = (float *)(size_t)131072; // never read here

static sconv_csr *make(const sconv_desc &d, double density, const sconv_plan *plan = nullptr)
{
    std::vector<float> w((size_t)d.K * (d.C / d.groups) * d.R * d.S);
    uint32_t s = 12345;
    for (float &v : w) {
        s = s * 1664525u + 1013904223u;
        v = (s >> 8) < density * (1 << 24) ? 0.5f + (float)(s & 0xff) : 0.f;
    }
    sconv_csr *h = nullptr;
    if (sconv_create_csr(&d, w.data(), plan, &h) != SCONV_OK) std::abort();
    return h;
}

static std::string forward(sconv_csr *h, int N)
{
    launched.clear();
    const int rc = sconv_forward(h, in, out, N, nullptr);
    return rc ? sconv_strerror(rc) : launched;
}

static std::string noalloc(sconv_csr *h, int N)
{
    launched.clear();
    const int rc = sconv_forward_noalloc(h, in, out, N, nullptr);
    return rc ? sconv_strerror(rc) : launched;
}

static std::string fc(sconv_csr *h, int N)
{
    launched.clear();
    const int rc = sconv_fc_forward(h, in, out, N, nullptr, 0, nullptr);
    return rc ? sconv_strerror(rc) : launched;
}

static const sconv_desc MID = {32, 13, 13, 50, 3, 3, 1, 1, 2}, FC = {600, 1, 1, 300, 1, 1, 1, 0, 1};
// long rows: flat streams on the matrix cores at large batches
static const sconv_desc LONG = {128, 13, 13, 256, 3, 3, 1, 1, 1}, LONG2 = {64, 27, 27, 96, 3, 3, 2, 0, 1}, LONGER = {472, 12, 12, 356, 3, 3, 1, 1, 1};
static const char *const FLAT = "flat", *const FLAT2 = "flat+reduce";

// What a tuning call measured holds for its batch size however many others follow.
static void tuned()
{
    sconv_csr *h = make(FC, 0.2);
    CHECK(fc(h, 4) == "fc_gather", "untuned: %s", launched.c_str());
    cost = {{"flat", 5.f}};
    CHECK(sconv_fc_tune(h, in, out, 4, 8, nullptr) == SCONV_OK, "tune");
    CHECK(fc(h, 4) == "fc_gather", "tuned: %s", launched.c_str());
    for (int n = 8; n <= 8 + 4 * 70; n += 4) fc(h, n);
    CHECK(fc(h, 4) == "fc_gather", "tuned, 70 batch sizes later: %s", launched.c_str());
    sconv_destroy_csr(h);

    h = make(FC, 0.2);
    cost = {{"fc_gather", 50.f}, {"mfma", 50.f}};
    CHECK(sconv_fc_tune(h, in, out, 4, 8, nullptr) == SCONV_OK, "tune");
    sconv_plan before, after;
    CHECK(fc(h, 4) == FLAT || launched == FLAT2, "measured against the model: %s", launched.c_str());
    sconv_fc_plan(h, 4, &before);
    for (int n = 8; n <= 8 + 4 * 70; n += 4) fc(h, n);
    CHECK(fc(h, 4) == FLAT || launched == FLAT2, "measured against the model, 70 batch sizes later: %s", launched.c_str());
    sconv_fc_plan(h, 4, &after);
    CHECK(!std::memcmp(&before, &after, sizeof before), "the tuned plan");
    sconv_destroy_csr(h);

    h = make(MID, 0.15);
    CHECK(forward(h, 9) == "gather", "untuned: %s", launched.c_str());
    cost = {{"gather", 50.f}, {"mfma", 50.f}};
    CHECK(sconv_tune(h, in, out, 9, 8, nullptr) == SCONV_OK, "tune");
    CHECK(forward(h, 9) == FLAT || launched == FLAT2, "measured against the model: %s", launched.c_str());
    sconv_csr_info(h, nullptr, nullptr, nullptr, &before);
    for (int n = 10; n < 80; ++n) forward(h, n);
    CHECK(forward(h, 9) == FLAT || launched == FLAT2, "measured against the model, 70 batch sizes later: %s", launched.c_str());
    sconv_csr_info(h, nullptr, nullptr, nullptr, &after);
    CHECK(!std::memcmp(&before, &after, sizeof before), "the tuned plan");
    sconv_destroy_csr(h);
    cost.clear();
}

// Without tuning the choice for a batch size does not depend on what ran before.
static void untuned()
{
    sconv_csr *h = make(MID, 0.15), *f = make(FC, 0.2);
    std::map<int, std::string> conv_first, fc_first;
    for (int round = 0; round < 2; ++round)
        for (int n = 1; n <= 150; ++n) {
            const std::string c = forward(h, n), g = fc(f, 4 * n);
            if (round == 0) {
                conv_first[n] = c;
                fc_first[n] = g;
            }
            CHECK(c == conv_first[n], "N=%d: %s, at first %s", n, c.c_str(), conv_first[n].c_str());
            CHECK(g == fc_first[n], "fc N=%d: %s, at first %s", 4 * n, g.c_str(), fc_first[n].c_str());
        }
    sconv_destroy_csr(h);
    sconv_destroy_csr(f);
}

// sconv_forward_noalloc takes every batch size that sconv_forward ran, and those that share its tiling (1 to 4), and
// launches what sconv_forward launches for it.
static void prepared()
{
    for (int first = 1; first <= 4; ++first) {
        sconv_csr *h = make(MID, 0.15), *again = make(MID, 0.15);
        forward(h, first);
        for (int n = 1; n <= 4; ++n) {
            const std::string got = noalloc(h, n), want = forward(again, n);
            CHECK(got == want, "prepared with N=%d, called with %d: %s instead of %s", first, n, got.c_str(), want.c_str());
        }
        sconv_destroy_csr(h);
        sconv_destroy_csr(again);
    }
    sconv_csr *h = make(MID, 0.15);
    CHECK(forward(h, 8) == "gather", "%s", launched.c_str());
    for (int n = 1; n <= 4; ++n) forward(h, n);
    for (int n = 9; n <= 68; ++n) {
        forward(h, n); // 64 tilings are remembered: that of the first plan, of 4 and of 8 to 68
        CHECK(noalloc(h, 8) == "gather", "with %d batch sizes since: %s", n - 4, launched.c_str());
    }
    sconv_destroy_csr(h);
}

// A call whose kernel's arrays find no room on the device runs on the flat-stream kernel, as it would without that kernel,
// and the arrays of other kernels stay.
static void no_room()
{
    for (int ok = 0; ok < 2; ++ok) {
        sconv_csr *h = make(MID, 0.15);
        uploads_ok = ok;
        uploads_fail = 1;
        CHECK(forward(h, 9) == FLAT || launched == FLAT2, "%d uploads, then none: %s", ok, launched.c_str());
        CHECK(forward(h, 9) == FLAT || launched == FLAT2, "again: %s", launched.c_str());
        CHECK(forward(h, 10) == "gather", "another batch size, room again: %s", launched.c_str());
        sconv_destroy_csr(h);
        h = make(FC, 0.2);
        uploads_ok = ok;
        uploads_fail = 1;
        CHECK(fc(h, 4) == FLAT || launched == FLAT2, "fc, %d uploads, then none: %s", ok, launched.c_str());
        sconv_destroy_csr(h);
    }
    const sconv_desc wide = {64, 13, 13, 64, 3, 3, 1, 1, 1};
    sconv_csr *h = make(wide, 0.6);
    CHECK(forward(h, 1) == "gather", "%s", launched.c_str());
    uploads_ok = 2; // (of the matrix-core kernel's three)
    uploads_fail = 1;
    const std::string got = forward(h, 64);
    CHECK(got == FLAT || got == FLAT2, "no room for the matrix-core arrays: %s", got.c_str());
    uploads_fail = 1000;
    CHECK(forward(h, 1) == "gather" && noalloc(h, 1) == "gather", "the gather arrays: %s", launched.c_str());
    uploads_fail = 0;
    CHECK(forward(h, 65) == "mfma", "room again: %s", launched.c_str());
    sconv_destroy_csr(h);
}

// A few short rows are summed apart; a layer of many of them, or with a weight that three bf16 parts do not hold, stays on
// the sparse kernels.
static void short_rows()
{
    const sconv_desc d = {64, 13, 13, 64, 3, 3, 1, 1, 1};
    for (int n_short = 0; n_short <= 8; ++n_short)
        for (int nnz = 0; nnz <= 4; ++nnz) {
            std::vector<int32_t> rowptr(1, 0), col;
            for (int k = 0; k < 64; ++k) {
                const int n = k % 8 == 1 && k / 8 < n_short ? nnz : 400;
                for (int j = 0; j < n; ++j) col.push_back(j);
                rowptr.push_back((int32_t)col.size());
            }
            std::vector<float> val(col.size(), 1.5f);
            sconv_csr *h = nullptr;
            if (sconv_create_csr_from_arrays(&d, rowptr.data(), col.data(), val.data(), nullptr, &h) != SCONV_OK) std::abort();
            const bool many = nnz > 0 && nnz < SCONV_MFMA_SHORT_ROW && n_short * SCONV_MFMA_SHORT_SHARE > 64;
            CHECK((forward(h, 64) == "mfma") == !many, "%d rows of %d: %s", n_short, nnz, launched.c_str());
            sconv_destroy_csr(h);
        }
}

static bool unpacks(sconv_csr *h, int which)
{
    int64_t n = 0;
    sconv_csr_info(h, &n, nullptr, nullptr, nullptr);
    std::vector<int32_t> ptr[2], off[2];
    std::vector<float> val[2];
    for (int i = 0; i < 2; ++i) {
        ptr[i].resize(4096);
        off[i].resize(n);
        val[i].resize(n);
        const int rc = i ? sconv_csr_unpack(h, which, ptr[i].data(), off[i].data(), val[i].data(), &n)
                         : sconv_csr_export(h, ptr[i].data(), off[i].data(), val[i].data(), &n);
        if (rc) return false;
    }
    return ptr[0] == ptr[1] && off[0] == off[1] && val[0] == val[1];
}

// A call that another kernel serves leaves its tiling unpacked: reported as ever, packed by the first call that runs it.
static void unpacked_tilings()
{
    sconv_csr *h = make(MID, 0.15);
    sconv_plan plan, want;
    int32_t count;
    packs = 0;
    CHECK(forward(h, 9) == "gather" && forward(h, 20) == "gather" && forward(h, 9) == "gather" && packs == 0, "%d packings", packs);
    sconv_csr_info(h, nullptr, nullptr, nullptr, &plan);
    sconv_rank_plans(h, 9, 1, &want, &count);
    CHECK(!std::memcmp(&plan, &want, sizeof plan), "the plan for 9 images");
    sconv_balance b;
    CHECK(unpacks(h, 1) && sconv_csr_balance(h, &b) == SCONV_OK && b.stream_entries >= b.nnz, "arrays on request");
    packs = 0;
    CHECK(forward(h, 1) == "gather" && packs == 1, "%d packings for batches of 1 to 4", packs);
    cost = {{"gather", 50.f}, {"mfma", 50.f}};
    sconv_tune(h, in, out, 9, 1, nullptr);
    cost.clear();
    packs = 0;
    CHECK((forward(h, 9) == FLAT || launched == FLAT2) && packs == 0, "after tuning: %s, %d packings", launched.c_str(), packs);
    for (int n = 10; n < 20; ++n) forward(h, n);
    CHECK(forward(h, 9) == FLAT || launched == FLAT2, "%s", launched.c_str());
    CHECK(unpacks(h, 1), "the arrays of 9 images");
    sconv_destroy_csr(h);
    h = make(MID, 0.15);
    packs = 0;
    uploads_fail = 1;
    CHECK((forward(h, 9) == FLAT || launched == FLAT2) && packs == 1, "no room: %s, %d packings", launched.c_str(), packs);
    sconv_destroy_csr(h);

    h = make(FC, 0.2);
    packs = uploads_fail = 0;
    CHECK(fc(h, 4) == "fc_gather" && fc(h, 8) == "fc_gather" && fc(h, 4) == "fc_gather" && packs == 0, "fc: %d packings", packs);
    CHECK(unpacks(h, 3), "fc: arrays on request");
    packs = 0;
    CHECK(sconv_fc_plan(h, 4, &plan) == SCONV_OK && packs == 1 && unpacks(h, 3), "fc: planned on request, %d packings", packs);
    sconv_destroy_csr(h);
    h = make(FC, 0.2);
    packs = 0;
    uploads_fail = 1;
    CHECK((fc(h, 12) == FLAT || launched == FLAT2) && packs == 1, "fc, no room: %s, %d packings", launched.c_str(), packs);
    sconv_destroy_csr(h);
}

// The first call with a batch size uploads what it reads and no more.
static void first_call()
{
    const sconv_desc d = {64, 13, 13, 64, 3, 3, 1, 1, 1};
    sconv_csr *h = make(d, 0.6);
    uploaded = 0;
    CHECK(forward(h, 64) == "mfma", "%s", launched.c_str());
    MfmaTiling t;
    choose_mfma(d, 64, t);
    const size_t fragments = ((size_t)t.n_tiles32 * t.total_steps + 1) * 3072, tables = 8u * (t.steps + t.steps_last);
    CHECK(uploaded == fragments + tables, "%zu bytes instead of %zu", uploaded, fragments + tables);
    uploaded = 0;
    forward(h, 64);
    forward(h, 65);
    CHECK(uploaded == 0, "%zu bytes once more", uploaded);
    sconv_destroy_csr(h);
}

// What sconv_route_of says is what the call launches.
static void routes()
{
    const char *const names[] = {"", "rows", "direct", "flat", "flat", "gather", "gather", "fc_gather", "mfma", "flat_mc"};
    bool seen[10] = {};
    auto check = [&](const sconv_route &r, const std::string &got, const sconv_desc &d, int N) {
        std::string want = r.kernel >= 1 && r.kernel <= 9 ? names[r.kernel] : "?";
        seen[r.kernel] = true;
        const bool lds = r.kernel == SCONV_KERNEL_ROWS || r.kernel == SCONV_KERNEL_FLAT || r.kernel == SCONV_KERNEL_FLOW;
        const bool parts = r.splits > 1 && (lds || r.kernel == SCONV_KERNEL_MFMA || r.kernel == SCONV_KERNEL_FLAT_MC);
        if (lds && r.launches > 1 + parts) want = "phase+" + want;
        if (parts) want += "+reduce";
        CHECK(got == want, "C%d %dx%d K%d %dx%d stride %d pad %d N=%d: %s, by the route %s", d.C, d.H, d.W, d.K, d.R, d.S, d.stride, d.pad, N,
              got.c_str(), want.c_str());
    };
    const sconv_plan plans[] = {{}, {2}, {3}, {4}, {1, 4}, {1, 8}};
    for (int hw : {5, 13, 29})
        for (int r : {1, 3, 4})
            for (int stride = 1; stride <= 2; ++stride)
                for (int pad = 0; pad <= 1; ++pad)
                    for (double density : {0.05, 0.7})
                        for (const sconv_plan &p : plans) {
                            const sconv_desc d = {48, hw, hw, 40, r, r, stride, pad, 1};
                            std::vector<float> w((size_t)d.K * d.C * r * r, 0.f);
                            for (size_t i = 0; i < w.size(); ++i) w[i] = (i * 2654435761u >> 8 & 1023) < density * 1024 ? 1.f : 0.f;
                            sconv_csr *h = nullptr;
                            if (sconv_create_csr(&d, w.data(), &p, &h) != SCONV_OK) continue;
                            for (int N : {1, 3, 6, 40, 200}) {
                                sconv_route route;
                                const int rc = sconv_route_of(h, N, &route);
                                const std::string got = forward(h, N);
                                if (rc) CHECK(got == sconv_strerror(rc), "%s instead of %s", got.c_str(), sconv_strerror(rc));
                                else check(route, got, d, N);
                            }
                            sconv_destroy_csr(h);
                        }
    bool mc_parts = false;
    for (const sconv_desc &d : {LONG, LONG2, LONGER})
        for (double density : {0.12, 0.2, 0.95}) {
            sconv_csr *h = make(d, density);
            for (int N : {1, 8, 16, 34, 64, 100, 256}) {
                sconv_route route;
                if (sconv_route_of(h, N, &route)) std::abort();
                check(route, forward(h, N), d, N);
                mc_parts |= route.kernel == SCONV_KERNEL_FLAT_MC && route.splits > 1;
            }
            sconv_destroy_csr(h);
        }
    CHECK(mc_parts, "no call of the flat streams on the matrix cores splits the channels");
    for (double density : {0.02, 0.2, 0.9}) {
        sconv_csr *h = make(FC, density);
        for (int N : {4, 12, 64, 256, 1024, 2048, 5, 1028}) {
            sconv_route route;
            const int rc = sconv_fc_route_of(h, N, &route);
            const std::string got = fc(h, N);
            if (rc) CHECK(got == sconv_strerror(rc), "%s instead of %s", got.c_str(), sconv_strerror(rc));
            else check(route, got, FC, N);
        }
        sconv_destroy_csr(h);
    }
    for (int k = 1; k <= 9; ++k) CHECK(seen[k], "kernel %d takes none of the calls", k);
}

// The flat streams on the matrix cores: kept as measured, prepared for the call without allocation, left when their arrays find
// no room, uploaded once for all batch sizes.
static void flat_mc()
{
    const std::string MC = "flat_mc";
    sconv_csr *h = make(LONG, 0.2);
    CHECK(noalloc(h, 256) == sconv_strerror(SCONV_ERR_PLAN), "never run: %s", launched.c_str());
    CHECK(forward(h, 256) == MC && noalloc(h, 256) == MC, "%s", launched.c_str());
    uploaded = 0;
    CHECK(forward(h, 200) == MC && forward(h, 256) == MC && uploaded == 0, "%s, %zu bytes once more", launched.c_str(), uploaded);
    cost = {{MC, 50.f}, {"mfma", 50.f}};
    CHECK(sconv_tune(h, in, out, 256, 4, nullptr) == SCONV_OK && (forward(h, 256) == FLAT || launched == FLAT2), "measured against the model: %s", launched.c_str());
    CHECK(noalloc(h, 256) == FLAT || launched == FLAT2, "%s", launched.c_str());
    CHECK(forward(h, 200) == MC, "another batch size: %s", launched.c_str());
    cost = {{"flat", 50.f}, {"mfma", 50.f}};
    CHECK(sconv_tune(h, in, out, 256, 4, nullptr) == SCONV_OK && forward(h, 256) == MC, "measured: %s", launched.c_str());
    for (int n = 10; n < 80; ++n) forward(h, n);
    CHECK(forward(h, 256) == MC && noalloc(h, 256) == MC, "70 batch sizes later: %s", launched.c_str());
    cost.clear();
    sconv_destroy_csr(h);
    for (int ok = 0; ok < 4; ++ok) { // (its arrays go up in order)
        h = make(LONG, 0.2);
        uploads_ok = ok;
        uploads_fail = 1;
        CHECK(forward(h, 256) == FLAT || launched == FLAT2, "%d uploads, then none: %s", ok, launched.c_str());
        CHECK(forward(h, 256) == FLAT || launched == FLAT2, "again: %s", launched.c_str());
        CHECK(forward(h, 200) == MC, "another batch size, room again: %s", launched.c_str());
        sconv_destroy_csr(h);
        uploads_ok = uploads_fail = 0;
    }
    // parts come out of the handle's scratch, or the caller's
    h = make(LONGER, 0.95);
    CHECK(forward(h, 34) == "flat_mc+reduce" && noalloc(h, 34) == "flat_mc+reduce", "%s", launched.c_str());
    sconv_destroy_csr(h);
    const sconv_plan plan = {3};
    h = make(LONG, 0.2, &plan);
    CHECK(forward(h, 256) == FLAT || launched == FLAT2, "a kernel was asked for: %s", launched.c_str());
    sconv_destroy_csr(h);
}

static sconv_csr *rows_of(const sconv_desc &d, const std::vector<int> &nnz)
{
    const int cols = d.C / d.groups * d.R * d.S;
    std::vector<int32_t> rowptr(1, 0), col;
    for (int k = 0; k < d.K; ++k) {
        const int n = nnz[k % nnz.size()];
        for (int j = 0; j < n; ++j) col.push_back((int)((int64_t)j * cols / n));
        rowptr.push_back((int32_t)col.size());
    }
    std::vector<float> val(col.size(), 1.5f);
    sconv_csr *h = nullptr;
    if (sconv_create_csr_from_arrays(&d, rowptr.data(), col.data(), val.data(), nullptr, &h) != SCONV_OK) std::abort();
    return h;
}

// Calls that measured slower on a gather kernel stay on the flat-stream kernel: rows of very different lengths, a few
// workgroups more than CUs, many large workgroups of the fully connected kernel; and calls beside them that measured faster.
static void gather_limits()
{
    struct Conv {
        sconv_desc d;
        int N;
        std::vector<int> nnz;
        bool gather;
    };
    std::vector<int> uneven(32, 122), level(32, 163);
    uneven[7] = 1182;
    uneven[20] = 400;
    const std::vector<Conv> convs = {
        {{164, 9, 9, 323, 3, 3, 2, 1, 1}, 18, uneven, false},          // 47.6 us, flat-stream kernel 21.4
        {{164, 9, 9, 323, 3, 3, 2, 1, 1}, 18, level, true},
        {{216, 18, 18, 35, 3, 3, 1, 1, 1}, 5, {1419}, false},          // 280 workgroups: 27.0 us, 24.6
        {{216, 18, 18, 32, 3, 3, 1, 1, 1}, 5, {1419}, true},           // 256
        {{256, 13, 13, 384, 3, 3, 1, 1, 1}, 1, {230}, true},
        {{384, 13, 13, 256, 3, 3, 1, 1, 2}, 16, {140, 173, 200}, true},  // 22.7, 25.3
        {{39, 53, 53, 58, 3, 3, 1, 1, 1}, 59, {3, 4, 6}, true},          // 20.7, 22.6
        {{80, 7, 7, 152, 1, 1, 1, 0, 1}, 139, {1}, true},                // fours through the image, or through each row: 4.9, 8.6
        {{52, 7, 7, 103, 3, 3, 1, 1, 1}, 197, {5, 6, 7}, true},          // 5.5, 8.4
    };
    for (const Conv &c : convs) {
        sconv_csr *h = rows_of(c.d, c.nnz);
        const bool gather = forward(h, c.N) == "gather";
        CHECK(gather == c.gather, "C%d K%d N=%d: %s", c.d.C, c.d.K, c.N, launched.c_str());
        sconv_destroy_csr(h);
    }
    sconv_csr *h = rows_of({8763, 1, 1, 47, 1, 1, 1, 0, 1}, {2610});
    CHECK(fc(h, 1020) != "fc_gather", "47 rows, batch 1020 (64.0 us, flat-stream kernel 46.6): %s", launched.c_str());
    CHECK(fc(h, 64) == "fc_gather", "47 rows, batch 64: %s", launched.c_str());
    sconv_destroy_csr(h);
}

// Layers of one tap go to the matrix cores only where the sums come no further from the exact ones.
static void one_tap_limits()
{
    // images of one and two positions: the gather kernel that keeps its sums in 64 bits
    struct Conv {
        sconv_desc d;
        int N;
        double density;
    };
    for (const Conv &c : {Conv{{64, 1, 1, 1024, 1, 1, 1, 0, 1}, 512, 0.5}, {{64, 1, 2, 1024, 1, 1, 1, 0, 1}, 256, 0.5}}) {
        sconv_csr *h = make(c.d, c.density);
        CHECK(forward(h, c.N) == "gather", "C%d %dx%d K%d N=%d: %s", c.d.C, c.d.H, c.d.W, c.d.K, c.N, launched.c_str());
        sconv_destroy_csr(h);
    }
    // fully connected flat streams of 12 parts are further from the exact sums than one of up to 512 nonzeros, and closer than one of more may be
    sconv_csr *h = make({295, 1, 1, 253, 1, 1, 1, 0, 1}, 0.9);
    CHECK(fc(h, 712) == "mfma", "295 -> 253, batch 712: %s", launched.c_str());
    sconv_destroy_csr(h);
    h = make({1529, 1, 1, 1290, 1, 1, 1, 0, 1}, 0.36);
    CHECK(fc(h, 868) == FLAT2, "1529 -> 1290, batch 868: %s", launched.c_str());
    sconv_destroy_csr(h);
    // calls that measured slower on the column kernel stay (rows of few nonzeros, rows of one to three among them), others go
    struct Rows {
        sconv_desc d;
        int N;
        std::vector<int> nnz;
        bool column;
    };
    const std::vector<Rows> calls = {
        {{334, 26, 26, 118, 1, 1, 1, 0, 2}, 44, {7, 14, 15, 23}, false},      // 15.5 us on the gather kernel, 16.6
        {{129, 41, 41, 61, 1, 1, 1, 0, 1}, 46, {6, 13, 14, 20}, false},       // 18.1, 19.9
        {{98, 33, 33, 447, 1, 1, 1, 0, 1}, 10, {2, 81, 5, 9, 5, 9, 5, 9, 5, 9, 5, 9, 9, 9, 9, 9, 9, 9, 9, 9, 9, 9, 9, 9, 9, 9}, false}, // flat streams 18.5, 24.3
        {{113, 54, 54, 332, 1, 1, 1, 0, 1}, 5, {14, 25, 39, 23}, true},       // gather kernel 25.0, 17.0
        {{192, 28, 28, 64, 1, 1, 1, 0, 1}, 64, {58}, true},                   // 15.4
    };
    for (const Rows &c : calls) {
        sconv_csr *g = rows_of(c.d, c.nnz);
        const bool column = forward(g, c.N) == "mfma";
        CHECK(column == c.column, "C%d %dx%d K%d N=%d: %s", c.d.C, c.d.H, c.d.W, c.d.K, c.N, launched.c_str());
        sconv_destroy_csr(g);
    }
}

// Layers of one tap are the column kernel's on the matrix cores, all others the staged one's.
static void column_calls()
{
    // those of test_gpu_mfma_column.py
    for (const std::vector<int> &c : {std::vector<int>{15, 40, 40, 32, 1, 30}, {17, 40, 40, 32, 1, 30}, {32, 19, 23, 65, 1, 30}, {33, 9, 11, 65, 1, 80},
                                      {41, 31, 7, 97, 1, 60}, {96, 28, 28, 70, 2, 33}, {100, 21, 21, 129, 1, 23}, {202, 13, 13, 130, 2, 128}, {250, 11, 13, 64, 1, 150}}) {
        sconv_csr *h = make({c[0], c[1], c[2], c[3], 1, 1, 1, 0, c[4]}, 0.9);
        column = false;
        CHECK(forward(h, c[5]).compare(0, 4, "mfma") == 0 && column, "C%d %dx%d K%d: %s, column %d", c[0], c[1], c[2], c[3], launched.c_str(), column);
        sconv_destroy_csr(h);
    }
    for (const std::vector<int> &c : {std::vector<int>{100, 512, 1020}, {777, 1000, 1020}, {2050, 300, 260}, {140, 3000, 128}}) {
        sconv_csr *h = make({c[0], 1, 1, c[1], 1, 1, 1, 0, 1}, 0.9);
        column = false;
        CHECK(fc(h, c[2]).compare(0, 4, "mfma") == 0 && column, "fc %d -> %d, batch %d: %s, column %d", c[0], c[1], c[2], launched.c_str(), column);
        sconv_destroy_csr(h);
    }
    for (const sconv_desc &d : {sconv_desc{64, 13, 13, 64, 3, 3, 1, 1, 1}, sconv_desc{128, 14, 14, 128, 2, 1, 1, 0, 1}}) {
        sconv_csr *h = make(d, 0.7);
        column = true;
        CHECK(forward(h, 128).compare(0, 4, "mfma") == 0 && !column, "C%d %dx%d stride %d: %s, column %d", d.C, d.R, d.S, d.stride, launched.c_str(), column);
        sconv_destroy_csr(h);
    }
}

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "tuned") tuned();
    else if (what == "untuned") untuned();
    else if (what == "prepared") prepared();
    else if (what == "no_room") no_room();
    else if (what == "short_rows") short_rows();
    else if (what == "first_call") first_call();
    else if (what == "routes") routes();
    else if (what == "flat_mc") flat_mc();
    else if (what == "gather_limits") gather_limits();
    else if (what == "column_calls") column_calls();
    else if (what == "one_tap_limits") one_tap_limits();
    else if (what == "unpacked_tilings") unpacked_tilings();
    else return 2;
    std::printf("%ld failures\n", failures);
    return failures ? 1 : 0;
}
