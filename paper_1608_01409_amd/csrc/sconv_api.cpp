// The extern "C" surface of libsconv (see include/sconv.h) and the roofline model of Section 2.2.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <iterator>
#include <limits>
#include <map>
#include <new>
#include <utility>
#include <vector>

#include "sconv_internal.h"

using namespace sconv;

// An earlier packing of a handle, kept with its device copies: a caller that alternates between batch sizes
// gets it back instead of packing and uploading again.
struct StashedPacking {
    bool flat = false;
    PackedLds lds;
    PackedFlat lds_flat;
    DeviceLds dev;
    bool uploaded = false;
    // fully connected packings only
    int fc_n = 0, fc_tiles = 0;
    sconv_desc fc_desc;
};
static const size_t kStashed = 3; // packings kept besides the current one

static void release_arrays(DeviceLds &dev)
{
    release(dev.pairs);
    release(dev.seg_ptr);
    release(dev.row_of);
    release(dev.store_tbl);
    dev = DeviceLds();
}

struct sconv_csr {
    sconv_desc desc;
    Canonical canon;
    sconv_plan requested;    // what the caller asked for (zeros = choose)
    bool has_lds = false;    // one of the two LDS packings below is filled
    bool flat = false;       // ... the flat-stream one
    PackedLds lds;
    PackedFlat lds_flat;
    PackedDirect direct;
    DeviceLds dev_lds;
    DeviceDirect dev_direct;
    bool lds_uploaded = false, direct_uploaded = false;
    int planned_n = 0;       // batch size the current LDS tiling was chosen for
    struct Planned {
        sconv_plan plan;
        double us;           // the cost model's time for it
        int phase_cg;        // as in LdsTiling
        bool tuned;          // measured by sconv_tune / sconv_fc_tune: kept, the others make room for later batch sizes
    };
    std::map<int, Planned> plan_of_n;        // tilings already chosen, by batch size
    // which kernel serves a batch size (by the cost models, or as measured): the flat-stream kernel with its plan,
    // the gather kernel (small launches), the matrix-core kernel (rather dense layers) or the flat streams on the matrix cores
    enum Kind { kLds, kGather, kMfma, kFlatMc };
    struct Choice {
        Kind kind;
        GatherShape gather;                  // t = 0: the gather kernel cannot take it
        MfmaTiling mfma;                     // mt = 0: the matrix-core kernel cannot take it
        FlatMcTiling mc;                     // mt = 0: the flat streams stay on the vector units
        bool tuned;                          // as in Planned
    };
    struct Alternatives {                    // for the convolution entry points, for the fully connected one
        std::map<int, Choice> choice_of_n;
        DeviceGather gather;
        DeviceMfma mfma;
    } conv_alt, fc_alt;
    struct {                                 // convolutions on kFlatMc
        DeviceLds dev;
        FlatMcTiling packed;                 // as packed; nt and splits follow the batch size
        bool uploaded = false;
    } flat_mc;
    int max_row_nnz = 0;
    int shortest_row = 0;                    // of the rows that are not empty
    bool mc_ok = false;                      // rows and weights are such that the flat streams may run on the matrix cores
    bool split_exact = true;                 // every weight is exactly three bf16 parts
    int short_rows = 0;                      // rows of 1 to SCONV_MFMA_SHORT_ROW - 1 nonzeros
    std::vector<StashedPacking> stash;       // earlier packings, oldest first
    // the layer the LDS kernels run: the layer itself, or for stride > 1 its stride-1 form over phase images
    bool phased = false;
    sconv_desc kdesc;
    Canonical kcanon;        // filled only when phased
    void *phase_buf = nullptr;
    size_t phase_bytes = 0;
    void *part_buf = nullptr; // partial results of launches that split the channels over workgroups
    size_t part_bytes = 0;
    const Canonical &kc() const { return phased ? kcanon : canon; }
    // real channels per phase of a group when the phase images can be picked out of the caller's input while
    // staging (a strided layer without padding), else 0
    int phase_cg() const { return (phased && desc.pad == 0) ? desc.C / desc.groups : 0; }
    // fully connected use (sconv_fc_forward): the layer as a 1x1 convolution whose positions are the batch
    int fc_n = 0;            // batch size the arrays below were packed for
    int fc_tiles = 0;        // the batch is cut into this many tiles of fc_n / fc_tiles images
    sconv_desc fc_desc;
    PackedFlat fc_flat;
    DeviceLds fc_dev;
    bool fc_uploaded = false;
    std::vector<StashedPacking> fc_stash;
    std::map<int, Planned> fc_plan_of_n;     // tilings sconv_fc_tune chose, by batch size
    size_t stash_cap = kStashed;             // packings kept besides the current one (more while tuning)
    int hip_err = 0;
};

static double avg_row_nnz(const sconv_csr *h) { return h->desc.K ? (double)h->canon.val.size() / h->desc.K : 0.0; }

static const LdsTiling &f_tiling(const sconv_csr *h) { return h->lds_flat.t; }

// Scratch owned by the handle, grown on demand.
static int grow(void **buf, size_t *have, size_t need, int *hip_err)
{
    if (need <= *have) return SCONV_OK;
    release(*buf);
    *buf = nullptr;
    *have = 0;
    const int rc = upload(nullptr, need, buf, hip_err);
    if (rc) return rc;
    *have = need;
    return SCONV_OK;
}

// A fixed piece of device memory handed out front to back (the entry point that must not allocate).
struct Workspace {
    char *base = nullptr;
    size_t bytes = 0, used = 0;
    void *take(size_t need)
    {
        const size_t at = (used + 255) & ~(size_t)255;
        if (at + need > bytes) return nullptr;
        used = at + need;
        return base + at;
    }
};

// Room for partial results: scratch the handle owns and grows, or a piece of `ws` when one is given.
static int take_parts(sconv_csr *h, size_t need, Workspace *ws, float **parts)
{
    if (ws) {
        *parts = static_cast<float *>(ws->take(need));
        return *parts ? SCONV_OK : SCONV_ERR_CAPACITY;
    }
    const int rc = grow(&h->part_buf, &h->part_bytes, need, &h->hip_err);
    *parts = rc ? nullptr : static_cast<float *>(h->part_buf);
    return rc;
}

// The flat-stream kernel and, when the tiling splits the channels, the reduction of its partial results.
// The partial results go to scratch the handle owns and grows, or into `ws` when one is given.
static int run_flat(sconv_csr *h, const sconv_desc &kd, const LdsTiling &t, const DeviceLds &dev, const Lds2Layout &lay,
                    const float *in, float *out, int n_kernel, int64_t rows, int64_t inner, const Epilogue &ep, void *stream,
                    Workspace *ws = nullptr)
{
    if (t.p.splits <= 1) return launch_lds2(kd, t, dev, lay, in, out, n_kernel, ep, 0, stream, &h->hip_err);
    const int64_t total = rows * inner;
    float *parts;
    int rc = take_parts(h, (size_t)total * t.p.splits * sizeof(float), ws, &parts);
    if (rc) return rc;
    rc = launch_lds2(kd, t, dev, lay, in, parts, n_kernel, ep, total, stream, &h->hip_err);
    if (rc) return rc;
    return launch_reduce(parts, out, t.p.splits, rows, inner, h->desc.K, ep, stream, &h->hip_err);
}

static bool same_plan(const sconv_plan &a, const sconv_plan &b)
{
    return a.kernel == b.kernel && a.nt == b.nt && a.cb == b.cb && a.waves == b.waves && a.cg == b.cg &&
           a.rows_w == b.rows_w && a.t == b.t && a.band == b.band && a.strip == b.strip && a.splits == b.splits;
}

// Choose (or re-choose) the LDS tiling for batch size n and pack for it.  The best tiling depends on the
// batch: with few image tiles smaller workgroups are needed to occupy every CU.  The handle changes only
// once the new packing exists: after an error it still holds, and runs, the packing it had.
static const size_t kPlansRemembered = 64; // batch sizes whose untuned tiling is kept; beyond that the table starts over

template <class Map>
static void drop_untuned(Map &of_n)
{
    for (auto it = of_n.begin(); it != of_n.end();) it = it->second.tuned ? std::next(it) : of_n.erase(it);
}

// Room for one more batch size: from kPlansRemembered untuned entries on they all go, tuned ones stay.  True if they went.
template <class Map>
static bool make_room(Map &of_n)
{
    size_t untuned = 0;
    for (const auto &e : of_n) untuned += !e.second.tuned;
    if (untuned < kPlansRemembered) return false;
    drop_untuned(of_n);
    return true;
}

static void remember_tiling(sconv_csr *h, int n, const LdsTiling &t)
{
    // a convolution's kernel choices go with its tilings: while one is remembered so is the other
    if (make_room(h->plan_of_n)) drop_untuned(h->conv_alt.choice_of_n);
    h->plan_of_n[n] = {t.p, t.us, t.phase_cg, false};
}

// The arrays of a tiling are there (a tiling that other kernels serve so far is not packed).
static bool is_packed(const PackedFlat &f) { return !f.seg.empty(); }

// The arrays of f's tiling: f itself, or packed into `own`.
static int packed(const sconv_desc &d, const Canonical &c, const PackedFlat &f, PackedFlat &own, const PackedFlat **out)
{
    *out = &f;
    if (is_packed(f)) return SCONV_OK;
    *out = &own;
    return pack_flat(d, c, f.t, own);
}

static int pack_now(const sconv_desc &d, const Canonical &c, PackedFlat &f)
{
    PackedFlat own;
    const PackedFlat *p;
    const int rc = packed(d, c, f, own, &p);
    if (!rc && p == &own) f = std::move(own);
    return rc;
}

// kPackLater: the tiling alone, its arrays with the first call that runs it.  kResidentOnly: for callers that must not allocate.
enum PackWhen { kPackNow, kPackLater, kResidentOnly };

static int plan_lds(sconv_csr *h, int n, PackWhen when = kPackNow)
{
    const bool resident_only = when == kResidentOnly;
    const sconv_desc &d = h->kdesc;
    const double avg = d.K ? (double)h->canon.val.size() / d.K : 0.0;
    LdsTiling t;
    int rc;
    auto known = h->plan_of_n.find(n);
    const bool fresh = known == h->plan_of_n.end();
    if (fresh && resident_only) return SCONV_ERR_PLAN; // never planned for this batch size
    rc = make_lds_tiling(d, fresh ? h->requested : known->second.plan, n, avg, t, h->phase_cg()); // a known tiling has every field: no search
    if (rc) return rc;
    auto remember = [&]() {
        if (fresh) remember_tiling(h, n, t);
    };
    if (h->has_lds && same_plan(t.p, h->flat ? h->lds_flat.t.p : h->lds.t.p)) {
        rc = h->flat && when == kPackNow ? pack_now(d, h->kc(), h->lds_flat) : SCONV_OK;
        if (rc) return rc;
        remember();
        h->planned_n = n;
        return SCONV_OK;
    }
    // an earlier packing for this tiling, device copies and all?
    size_t found = h->stash.size();
    for (size_t i = 0; i < h->stash.size(); ++i) {
        const StashedPacking &sp = h->stash[i];
        if (same_plan(t.p, sp.flat ? sp.lds_flat.t.p : sp.lds.t.p)) found = i;
    }
    StashedPacking next;
    if (found < h->stash.size()) {
        StashedPacking &sp = h->stash[found];
        if (resident_only && !sp.uploaded) return SCONV_ERR_PLAN;
        rc = sp.flat && when == kPackNow ? pack_now(d, h->kc(), sp.lds_flat) : SCONV_OK;
        if (rc) return rc;
        next = std::move(h->stash[found]);
        h->stash.erase(h->stash.begin() + (long)found);
    } else if (resident_only) {
        return SCONV_ERR_PLAN; // the packing for this tiling has been dropped: it would have to be built and uploaded
    } else {
        next.flat = is_flat_kernel(t.p.kernel);
        if (next.flat && when == kPackLater)
            next.lds_flat.t = t;
        else
            rc = next.flat ? pack_flat(d, h->kc(), t, next.lds_flat) : pack_lds(d, h->kc(), t, next.lds);
        if (rc) return rc;
    }
    if (h->has_lds) { // set the current packing aside
        StashedPacking old;
        old.flat = h->flat;
        old.lds = std::move(h->lds);
        old.lds_flat = std::move(h->lds_flat);
        old.dev = h->dev_lds;
        old.uploaded = h->lds_uploaded;
        h->stash.push_back(std::move(old));
        // (resident_only: one packing left the stash and one entered it, so nothing has to go, and nothing may:
        // hipFree is not for that caller)
        while (!resident_only && h->stash.size() > h->stash_cap) { // hipFree waits for launches that still read the arrays
            release_arrays(h->stash.front().dev);
            h->stash.erase(h->stash.begin());
        }
    }
    h->flat = next.flat;
    h->lds = std::move(next.lds);
    h->lds_flat = std::move(next.lds_flat);
    h->dev_lds = next.dev;
    h->lds_uploaded = next.uploaded;
    h->has_lds = true;
    remember();
    h->planned_n = n;
    return SCONV_OK;
}

static int finish_create(sconv_csr *h, const sconv_plan *plan)
{
    std::memset(&h->requested, 0, sizeof(h->requested));
    if (plan) h->requested = *plan;
    if (h->requested.kernel < 0 || h->requested.kernel > 4) return SCONV_ERR_PLAN;
    const sconv_desc &d = h->desc;
    for (int k = 0; k < d.K; ++k) {
        const int nnz = h->canon.rowptr[k + 1] - h->canon.rowptr[k];
        h->max_row_nnz = std::max(h->max_row_nnz, nnz);
        h->short_rows += nnz > 0 && nnz < SCONV_MFMA_SHORT_ROW;
    }
    for (float v : h->canon.val) h->split_exact = h->split_exact && mfma_weight_ok(v);
    h->shortest_row = shortest_row(h->canon);
    h->mc_ok = flat_mc_weights_ok(d, h->canon);
    int rc = pack_direct(d, h->canon, h->direct);
    if (rc) return rc;
    h->kdesc = d;
    if (d.stride > 1 && h->requested.kernel != 2) {
        // phase images; layers whose virtual form is out of range keep the direct kernel
        sconv_desc v;
        phase_desc(d, v);
        if (validate_desc(v) == SCONV_OK && phase_canonical(d, h->canon, h->kcanon) == SCONV_OK) {
            h->kdesc = v;
            h->phased = true;
        }
    }
    if (h->requested.kernel != 2 && (d.stride == 1 || h->phased)) {
        // tuned for a large batch until the first forward call says otherwise; small ones go to the direct kernel
        rc = plan_lds(h, h->requested.nt ? h->requested.nt : 256);
        if (rc != SCONV_OK && h->requested.kernel != 0) return rc;
    } else if (h->requested.kernel == 1 || is_flat_kernel(h->requested.kernel)) {
        return SCONV_ERR_PLAN;
    }
    return SCONV_OK;
}

extern "C" int sconv_create_csr(const sconv_desc *desc, const float *dense_w, const sconv_plan *plan, sconv_csr **out)
{
    if (!desc || !dense_w || !out) return SCONV_ERR_NULL;
    *out = nullptr;
    int rc = validate_desc(*desc);
    if (rc) return rc;
    sconv_csr *h = new (std::nothrow) sconv_csr();
    if (!h) return SCONV_ERR_NOMEM;
    try {
        h->desc = *desc;
        rc = build_canonical_from_dense(*desc, dense_w, h->canon);
        if (!rc) rc = finish_create(h, plan);
    } catch (const std::bad_alloc &) {
        rc = SCONV_ERR_NOMEM;
    }
    if (rc) {
        delete h;
        return rc;
    }
    *out = h;
    return SCONV_OK;
}

extern "C" int sconv_create_csr_from_arrays(const sconv_desc *desc, const int32_t *rowptr, const int32_t *colidx,
                                            const float *values, const sconv_plan *plan, sconv_csr **out)
{
    if (!desc || !rowptr || !out) return SCONV_ERR_NULL;
    *out = nullptr;
    int rc = validate_desc(*desc);
    if (rc) return rc;
    sconv_csr *h = new (std::nothrow) sconv_csr();
    if (!h) return SCONV_ERR_NOMEM;
    try {
        h->desc = *desc;
        rc = build_canonical_from_arrays(*desc, rowptr, colidx, values, h->canon);
        if (!rc) rc = finish_create(h, plan);
    } catch (const std::bad_alloc &) {
        rc = SCONV_ERR_NOMEM;
    }
    if (rc) {
        delete h;
        return rc;
    }
    *out = h;
    return SCONV_OK;
}

extern "C" int sconv_lower_offsets(const sconv_desc *desc, int32_t layout, const int32_t *rowptr, const int32_t *colidx,
                                   int32_t *off, int32_t *step_y, int32_t *step_x)
{
    if (!desc || !rowptr) return SCONV_ERR_NULL;
    int rc = validate_desc(*desc);
    if (rc) return rc;
    if (layout != SCONV_LAYOUT_CHW && layout != SCONV_LAYOUT_HWC) return SCONV_ERR_DESC;
    rc = validate_csr(*desc, rowptr, colidx);
    if (rc) return rc;
    if (rowptr[desc->K] > 0 && !off) return SCONV_ERR_NULL;
    lower_offsets(*desc, layout, rowptr, colidx, off);
    const Geometry g = geometry(*desc);
    const int per_x = layout == SCONV_LAYOUT_HWC ? desc->C : 1;
    if (step_y) *step_y = desc->stride * g.Wp * per_x;
    if (step_x) *step_x = desc->stride * per_x;
    return SCONV_OK;
}

extern "C" int sconv_csr_info(const sconv_csr *h, int64_t *nnz, int32_t *out_h, int32_t *out_w, sconv_plan *plan)
{
    if (!h) return SCONV_ERR_NULL;
    const Geometry g = geometry(h->desc);
    if (nnz) *nnz = (int64_t)h->canon.val.size();
    if (out_h) *out_h = g.OH;
    if (out_w) *out_w = g.OW;
    if (plan) {
        std::memset(plan, 0, sizeof(*plan));
        if (h->has_lds)
            *plan = h->flat ? h->lds_flat.t.p : h->lds.t.p;
        else
            plan->kernel = 2;
    }
    return SCONV_OK;
}

extern "C" int sconv_csr_balance(const sconv_csr *h, sconv_balance *out)
{
    if (!h || !out) return SCONV_ERR_NULL;
    if (!h->has_lds || !h->flat) return SCONV_ERR_PLAN;
    PackedFlat own;
    const PackedFlat *arrays;
    try {
        const int rc = packed(h->kdesc, h->kc(), h->lds_flat, own, &arrays);
        if (rc) return rc;
    } catch (const std::bad_alloc &) {
        return SCONV_ERR_NOMEM;
    }
    const PackedFlat &f = *arrays;
    const LdsTiling &t = f.t;
    std::memset(out, 0, sizeof(*out));
    out->nnz = (int64_t)h->canon.val.size();
    const int n_wg = t.wave_slots / t.rg; // groups * nkt workgroups' worth of row tiles
    double wg_sum = 0, wg_max = 0;
    for (int wg = 0; wg < n_wg; ++wg) {
        double wg_total = 0;
        for (int b = 0; b < t.nblk; ++b) {
            double sum = 0, mx = 0, simd[4] = {0, 0, 0, 0};
            int on_simd[4] = {0, 0, 0, 0};
            for (int r = 0; r < t.rg; ++r) {
                const uint32_t word = f.seg[((size_t)(wg * t.rg + r) * t.nblk + b) * 2 + 1];
                const double ch = (word & 0x7fffffffu) - ((word >> 31) ? 0.5 : 0.0); // a half chunk counts as half
                out->stream_entries += (int64_t)(ch * SCONV_FLAT_CHUNK + 0.5);
                sum += ch;
                mx = std::max(mx, ch);
                // the cg waves of a row group run the same stream; wave index = r * cg + column group
                for (int c = 0; c < t.p.cg; ++c) {
                    simd[(r * t.p.cg + c) & 3] += ch;
                    on_simd[(r * t.p.cg + c) & 3]++;
                }
            }
            double smx = 0;
            for (int q = 0; q < 4; ++q)
                if (on_simd[q]) smx = std::max(smx, simd[q] / on_simd[q]);
            out->wave_mean += sum / t.rg;
            out->wave_max += mx;
            out->simd_max += smx;
            wg_total += mx;
        }
        wg_sum += wg_total;
        wg_max = std::max(wg_max, wg_total);
    }
    out->workgroup_mean = n_wg ? wg_sum / n_wg : 0;
    out->workgroup_max = wg_max;
    return SCONV_OK;
}

static Canonical fc_canonical(const sconv_csr *h, const sconv_desc &kd);

static int export_canonical(const sconv_desc &d, const Canonical &c, int32_t *rowptr, int32_t *off, float *values,
                            int64_t *nnz_io)
{
    if (!nnz_io) return SCONV_ERR_NULL;
    const int64_t nnz = (int64_t)c.val.size();
    const int64_t cap = *nnz_io;
    *nnz_io = nnz;
    if (cap < nnz) return SCONV_ERR_CAPACITY;
    if (!rowptr || (nnz > 0 && (!off || !values))) return SCONV_ERR_NULL;
    std::memcpy(rowptr, c.rowptr.data(), sizeof(int32_t) * (d.K + 1));
    if (nnz) {
        std::memcpy(off, c.off.data(), sizeof(int32_t) * nnz);
        std::memcpy(values, c.val.data(), sizeof(float) * nnz);
    }
    return SCONV_OK;
}

extern "C" int sconv_csr_export(const sconv_csr *h, int32_t *rowptr, int32_t *off, float *values, int64_t *nnz_io)
{
    if (!h) return SCONV_ERR_NULL;
    return export_canonical(h->desc, h->canon, rowptr, off, values, nnz_io);
}

extern "C" int sconv_csr_unpack(const sconv_csr *h, int32_t which, int32_t *rowptr, int32_t *off, float *values,
                                int64_t *nnz_io)
{
    if (!h) return SCONV_ERR_NULL;
    Canonical c;
    PackedFlat own;
    const PackedFlat *arrays;
    int rc;
    try {
        if (which == 1) {
            if (!h->has_lds) return SCONV_ERR_PLAN;
            rc = h->flat ? packed(h->kdesc, h->kc(), h->lds_flat, own, &arrays) : SCONV_OK;
            if (!rc) rc = h->flat ? unpack_flat(h->kdesc, *arrays, c) : unpack_lds(h->kdesc, h->lds, c);
            if (!rc && h->phased) {
                Canonical real;
                rc = unphase_canonical(h->desc, c, real);
                c = std::move(real);
            }
        } else if (which == 2) {
            rc = unpack_direct(h->desc, h->direct, c);
        } else if (which == 3) {
            // the fully connected packing: offsets are feature * (positions per tile) in the wide image
            if (h->fc_n <= 0) return SCONV_ERR_PLAN;
            rc = packed(h->fc_desc, fc_canonical(h, h->fc_desc), h->fc_flat, own, &arrays);
            if (!rc) rc = unpack_flat(h->fc_desc, *arrays, c);
            if (!rc) {
                const int w = h->fc_desc.W;
                for (auto &o : c.off) {
                    if (o % w) return SCONV_ERR_CSR;
                    o /= w;
                }
            }
        } else {
            return SCONV_ERR_PLAN;
        }
    } catch (const std::bad_alloc &) {
        return SCONV_ERR_NOMEM;
    }
    if (rc) return rc;
    return export_canonical(h->desc, c, rowptr, off, values, nnz_io);
}

static int forward_impl(sconv_csr *h, const float *in, float *out, int32_t N, const Epilogue &ep, void *hip_stream,
                        Workspace *ws = nullptr);

extern "C" int sconv_forward(sconv_csr *h, const float *in, float *out, int32_t N, void *hip_stream)
{
    return forward_impl(h, in, out, N, Epilogue(), hip_stream);
}

extern "C" int sconv_forward_fused(sconv_csr *h, const float *in, float *out, int32_t N, const float *bias, int32_t relu,
                                   void *hip_stream)
{
    Epilogue ep;
    ep.bias = bias;
    ep.relu = relu != 0;
    return forward_impl(h, in, out, N, ep, hip_stream);
}

// No field of the tiling was requested: the library follows the batch size, and may leave the LDS kernels alone.
static bool free_choice(const sconv_csr *h)
{
    const sconv_plan &rq = h->requested;
    return !rq.nt && !rq.cb && !rq.waves && !rq.cg && !rq.rows_w && !rq.t && !rq.band && !rq.strip && !rq.splits;
}

// How far the matrix-core kernel's model is trusted against the flat-stream kernel's (GatherShape::margin for the gather
// kernels).  Of 4100 random calls it was chosen for, 7 take more than 2 % longer than on the flat-stream kernel (at most 14 %).
static const double kMfmaMargin = 1.15;
// The column kernel against a gather kernel, whose model reads high for short rows: of 120 random calls that left it at 1.25 13 took 2-18 %
// longer (1.25x on average); with the larger factor where rows have fewer than 16 nonzeros on average 4 of 97, 2-8 % (1.31x).
static const double kColumnGatherMargin = 1.25, kColumnGatherMarginShort = 1.45;
static const double kColumnShortRows = 16.0;

// The flat streams on the matrix cores against the same on the vector units and against the three-part kernel.  Of 357 random
// calls that went there from the former at 1.0, 12 took more than 2 % longer, two of them more than 10 %; at 1.01 it is 6 of 341,
// none more than 10 %, and at 1.03 one less, while 27 more stay that would gain 1.12x.  None of 47 from the latter was slower.
static const double kFlatMcMargin = 1.01, kFlatMcMfmaMargin = 1.15;
// Strided layers take longer on the vector units than their model says: 32 of them 1.09-2.2 times (stride 1: 1.06 on average).
static const double kFlatPhasedReadsLow = 1.09;

// The LDS path's time for N images: the flat-stream kernel's, and for layers that need phase images the pass that writes
// them (a launch, and their bytes written and read).
static double planned_us(const sconv_csr *h, int N, double flat_us, int phase_cg)
{
    if (!h->phased || flat_us <= 0 || phase_cg > 0) return flat_us;
    return flat_us + 4.0 + 2.0 * N * h->kdesc.C * h->kdesc.H * h->kdesc.W * 4.0 / 4.0e6;
}

// Which kernel a call with N images goes to; every kernel's cost model is asked, `lds_us` is the flat-stream path's time.
// Gather: launches with little arithmetic; its multiply-adds cost about three times the LDS kernels' (4.4 against 10-20
// million per microsecond), its fixed price is a third of theirs (3.5 us against 6-15).  Matrix cores: layers where the
// zeros they multiply cost less than what their rate wins.
static const sconv_csr::Choice &choose_kernel(sconv_csr *h, bool fc, int N, double lds_us, int lds_splits)
{
    sconv_csr::Alternatives &alt = fc ? h->fc_alt : h->conv_alt;
    auto known = alt.choice_of_n.find(N);
    if (known != alt.choice_of_n.end()) return known->second;
    sconv_csr::Choice c = {sconv_csr::kLds, {0, 0, 0.0, 0.0, 0.0}, {}, {}, false};
    double best = lds_us; // (a tiling the cost model gave no time keeps the call)
    if (fc ? fc_gather_fits(h->desc, N) : gather_fits(h->desc, N)) {
        c.gather = fc ? choose_fc_gather(h->desc, N, avg_row_nnz(h), h->max_row_nnz) : choose_gather(h->desc, N, avg_row_nnz(h), h->max_row_nnz);
        const double us = c.gather.us * c.gather.margin;
        if (us < best) {
            c.kind = sconv_csr::kGather;
            best = us;
        }
    }
    const sconv_csr::Kind without = c.kind;
    if (h->split_exact && h->short_rows * SCONV_MFMA_SHORT_SHARE <= h->desc.K && mfma_fits(h->desc, N, fc) && choose_mfma(h->desc, N, c.mfma)) {
        if (c.mfma.us * kMfmaMargin < best) c.kind = sconv_csr::kMfma;
    } else {
        c.mfma = MfmaTiling();
    }
    // The flat streams on the matrix cores, where the sums of no row are further from the exact ones than those they replace: what
    // counts is the length of the chains there, which parts make shorter.
    const int row = h->shortest_row;
    const bool three_parts = c.kind == sconv_csr::kMfma, flushed = three_parts || lds_splits > 1;
    const bool exact = three_parts ? row >= (c.mfma.splits <= 1 ? SCONV_MC_LONG_ROW : c.mfma.splits * SCONV_MC_LONG_ROW_SPLIT)
                                   : c.kind == sconv_csr::kLds && (lds_splits <= 1 || row >= lds_splits * SCONV_MC_ROW_SPLIT);
    if (!fc && exact && h->mc_ok && mfma_fits(h->desc, N, false) && choose_flat_mc(h->desc, h->canon, N, flushed, c.mc)) {
        if (three_parts ? c.mc.us * kFlatMcMfmaMargin < c.mfma.us : c.mc.us * kFlatMcMargin < lds_us * (h->phased ? kFlatPhasedReadsLow : 1.0)) c.kind = sconv_csr::kFlatMc;
    } else {
        c.mc = FlatMcTiling();
    }
    // Layers of one tap: the column kernel takes what the staged one would take, in no fewer parts, and of the rest what is faster there
    // with sums no further from the exact ones: the four-position gather kernel's of short rows (the other gather kernels keep theirs in
    // 64 bits: 64 -> 1024, 1x1 images, batch 512, rows of up to 41, 2.5e-8 where the matrix cores have 3.8e-8), the vector units' unless
    // they make many more parts.  Layers with short rows stay: each of those is a pass over a workgroup's positions that no model counts
    // (of 25 random calls that left with some, 9 took 2-49 % longer).  (Flat streams that are on the matrix cores stay there, also where the
    // column kernel is faster: 400 -> 64, 28x28, batch 100, density 0.3 takes 61.5 us, and would take 33.6.)
    if (c.mfma.one_tap) {
        const bool staged = c.kind == sconv_csr::kMfma, flat_mc = c.kind == sconv_csr::kFlatMc;
        const int parts = c.mfma.splits, chain_parts = SCONV_MFMA_CHAIN_PARTS * (h->max_row_nnz <= SCONV_MFMA_CHAIN_ROW ? 2 : 1);
        MfmaTiling m = c.mfma;
        bool can = choose_mfma_column(h->desc, N, staged || flat_mc ? parts : 1, m);
        const bool near = !h->short_rows && (c.kind == sconv_csr::kGather ? !fc && gather4_fits(h->desc) && h->max_row_nnz <= SCONV_MFMA_GATHER_ROW
                                                                          : lds_splits <= chain_parts * m.splits);
        const double margin = c.kind != sconv_csr::kGather ? kMfmaMargin : avg_row_nnz(h) < kColumnShortRows ? kColumnGatherMarginShort : kColumnGatherMargin;
        if (!staged && !near) can = choose_mfma_column(h->desc, N, parts, m);   // (for the tuner, as it was)
        c.mfma = can ? m : MfmaTiling();
        if (staged) c.kind = can ? sconv_csr::kMfma : without;
        else if (can && !flat_mc && near && m.us * margin < best) c.kind = sconv_csr::kMfma;
    }
    // What is left to the vector units after all that, the gather kernel of four positions takes with less of a margin.
    if (c.kind == sconv_csr::kLds && c.gather.flat_us > 0 && c.gather.flat_us < lds_us) c.kind = sconv_csr::kGather;
    if (fc) make_room(alt.choice_of_n); // (a convolution's choices make room with its tilings, in plan_lds)
    return alt.choice_of_n[N] = c;
}

// Set-up on this device: the address of the library's static scratch is looked up with the first upload, so that
// sconv_forward_noalloc finds it known (a failure here is that entry point's to report).
static void find_static_scratch()
{
    void *base;
    size_t bytes;
    int ignored = 0;
    (void)static_scratch(&base, &bytes, &ignored);
}

static int upload_direct(sconv_csr *h)
{
    if (h->direct_uploaded) return SCONV_OK;
    int rc = upload(h->direct.rowptr.data(), h->direct.rowptr.size() * 4, &h->dev_direct.rowptr, &h->hip_err);
    if (!rc) rc = upload(h->direct.trip.data(), h->direct.trip.size() * 4, &h->dev_direct.trip, &h->hip_err);
    if (rc) {
        release(h->dev_direct.rowptr);
        h->dev_direct = DeviceDirect();
        return rc;
    }
    h->direct_uploaded = true;
    return SCONV_OK;
}

static void release_gather(DeviceGather &dev)
{
    for (void *p : {dev.ent, dev.rowptr}) release(p);
    dev = DeviceGather();
}

static void release_mfma(DeviceMfma &dev)
{
    for (void *p : {dev.wfrag, dev.uoff, dev.choff}) release(p);
    dev = DeviceMfma();
}

static bool resident(const sconv_csr *h, const sconv_csr::Alternatives &alt, const sconv_csr::Choice &c)
{
    if (c.kind == sconv_csr::kFlatMc) return h->flat_mc.uploaded;
    return c.kind == sconv_csr::kGather ? alt.gather.uploaded : alt.mfma.uploaded && (!h->short_rows || h->direct_uploaded);
}

// Pack and upload what the chosen kernel reads (the same arrays for every batch size), once.
static int prepare_choice(sconv_csr *h, bool fc, const sconv_csr::Choice &c)
{
    sconv_csr::Alternatives &alt = fc ? h->fc_alt : h->conv_alt;
    if (resident(h, alt, c)) return SCONV_OK;
    int rc;
    if (c.kind == sconv_csr::kGather) {
        PackedGather p;
        rc = fc ? pack_fc_gather(h->desc, h->canon, p) : pack_gather(h->desc, h->canon, p);
        if (!rc) rc = upload(p.ent.data(), p.ent.size() * 8, &alt.gather.ent, &h->hip_err);
        if (!rc) rc = upload(p.rowptr.data(), p.rowptr.size() * 4, &alt.gather.rowptr, &h->hip_err);
        if (!rc) alt.gather.uploaded = true;
        else release_gather(alt.gather);
    } else if (c.kind == sconv_csr::kFlatMc) {
        PackedFlatMc p;
        DeviceLds &dev = h->flat_mc.dev;
        h->flat_mc.packed = c.mc;
        rc = pack_flat_mc(mfma_desc(h->desc), h->canon, h->flat_mc.packed, p);
        if (!rc) rc = upload(p.stream.data(), p.stream.size(), &dev.pairs, &h->hip_err);
        if (!rc) rc = upload(p.seg.data(), p.seg.size() * 4, &dev.seg_ptr, &h->hip_err);
        if (!rc) rc = upload(p.row_of.data(), p.row_of.size() * 4, &dev.row_of, &h->hip_err);
        if (!rc) rc = upload(p.choff.data(), p.choff.size() * 4, &dev.store_tbl, &h->hip_err);
        if (!rc) h->flat_mc.uploaded = true;
        else release_arrays(dev);
    } else {
        PackedMfma p;
        rc = alt.mfma.uploaded ? SCONV_OK : pack_mfma(h->desc, h->canon, c.mfma, p);
        if (!rc && !alt.mfma.uploaded) {
            rc = upload(p.wfrag.data(), p.wfrag.size() * 2, &alt.mfma.wfrag, &h->hip_err);
            if (!rc) rc = upload(p.uoff.data(), p.uoff.size() * 4, &alt.mfma.uoff, &h->hip_err);
            if (!rc) rc = upload(p.choff.data(), p.choff.size() * 4, &alt.mfma.choff, &h->hip_err);
            alt.mfma.short_rows = h->short_rows > 0;
            if (!rc) alt.mfma.uploaded = true;
        }
        if (!rc && h->short_rows) rc = upload_direct(h); // what the kernel sums short rows from
        if (rc) release_mfma(alt.mfma);
    }
    return rc;
}

// False if the chosen kernel's arrays cannot be had (no room for them beside the flat-stream kernel's): calls with N images
// then stay with the flat-stream kernel.
static bool ready(sconv_csr *h, bool fc, int N, const sconv_csr::Choice &c)
{
    int rc;
    try {
        rc = prepare_choice(h, fc, c);
    } catch (const std::bad_alloc &) {
        rc = SCONV_ERR_NOMEM;
    }
    if (rc) (fc ? h->fc_alt : h->conv_alt).choice_of_n[N].kind = sconv_csr::kLds;
    return rc == SCONV_OK;
}

// ws: as for run_flat
static int launch_choice(sconv_csr *h, bool fc, const sconv_csr::Choice &c, const float *in, float *out, int N, const Epilogue &ep,
                         void *stream, Workspace *ws = nullptr)
{
    const sconv_csr::Alternatives &alt = fc ? h->fc_alt : h->conv_alt;
    if (c.kind == sconv_csr::kGather)
        return fc ? launch_fc_gather(h->desc, alt.gather, c.gather, in, out, N, ep, stream, &h->hip_err)
                  : launch_gather(h->desc, alt.gather, c.gather, in, out, N, ep, stream, &h->hip_err);
    FlatMcTiling mc = h->flat_mc.packed;
    mc.nt = c.mc.nt;
    mc.splits = c.mc.splits;
    auto launch = [&](float *to, int64_t split_stride) {
        return c.kind == sconv_csr::kFlatMc ? launch_flat_mc(h->desc, mc, h->flat_mc.dev, in, to, N, ep, split_stride, stream, &h->hip_err)
                                            : launch_mfma(h->desc, c.mfma, alt.mfma, h->dev_direct, in, to, N, fc, ep, split_stride, stream, &h->hip_err);
    };
    const int splits = c.kind == sconv_csr::kFlatMc ? mc.splits : c.mfma.splits;
    if (splits <= 1) return launch(out, 0);
    const Geometry g = geometry(h->desc);
    const int64_t rows = fc ? h->desc.K : (int64_t)N * h->desc.K, inner = fc ? N : (int64_t)g.OH * g.OW;
    float *parts;
    int rc = take_parts(h, (size_t)(rows * inner) * splits * sizeof(float), ws, &parts);
    if (!rc) rc = launch(parts, rows * inner);
    return rc ? rc : launch_reduce(parts, out, splits, rows, inner, h->desc.K, ep, stream, &h->hip_err);
}

static int upload_flat(sconv_csr *h)
{
    if (h->lds_uploaded) return SCONV_OK;
    const PackedFlat &f = h->lds_flat;
    int rc = upload(f.pairs.data(), f.pairs.size() * 8, &h->dev_lds.pairs, &h->hip_err);
    if (!rc) rc = upload(f.seg.data(), f.seg.size() * 4, &h->dev_lds.seg_ptr, &h->hip_err);
    if (!rc) rc = upload(f.row_of.data(), f.row_of.size() * 4, &h->dev_lds.row_of, &h->hip_err);
    if (!rc) rc = upload(f.store_tbl.data(), f.store_tbl.size() * 4, &h->dev_lds.store_tbl, &h->hip_err);
    if (rc) return rc;
    h->lds_uploaded = true;
    return SCONV_OK;
}

// What the flat-stream path would keep in scratch for N images: partial results, phase images (256-byte pieces).
static size_t lds_scratch(const sconv_csr *h, int N, const sconv_csr::Planned &p)
{
    const Geometry g = geometry(h->desc);
    size_t parts = p.plan.splits > 1 ? (size_t)N * h->desc.K * g.OH * g.OW * p.plan.splits * sizeof(float) : 0;
    size_t phase = h->phased && p.phase_cg <= 0 ? (size_t)N * h->kdesc.C * h->kdesc.H * h->kdesc.W * sizeof(float) : 0;
    if (parts) phase = (phase + 255) & ~(size_t)255;
    return phase + parts;
}

// (batches below 4 use the tiling of batch 4: one tile of 4 images, not all of them present)
static int planned_batch(int N) { return N < 4 ? 4 : N; }

// The library decides which kernel a call goes to: no plan field was given, and the flat-stream kernel can take the layer.
static bool may_choose(const sconv_csr *h) { return h->has_lds && free_choice(h) && h->requested.kernel == 0 && h->flat; }

// Plans for a batch of N where the tiling follows it (only when none of its fields was requested), and sets *c to the kernel
// that takes the call instead of the handle's own, or to null.  The tiling is chosen either way, for its time; its arrays are
// packed if a call reads them.
static int decide(sconv_csr *h, int N, const sconv_csr::Choice **c)
{
    *c = nullptr;
    if (!h->has_lds || !free_choice(h)) return SCONV_OK;
    const int n_plan = planned_batch(N);
    PackWhen when = kPackNow;
    if (may_choose(h)) {
        auto planned = h->plan_of_n.find(n_plan);
        if (planned == h->plan_of_n.end()) {
            LdsTiling t;
            const int rc = make_lds_tiling(h->kdesc, h->requested, n_plan, avg_row_nnz(h), t, h->phase_cg());
            if (rc) return rc;
            remember_tiling(h, n_plan, t);
            planned = h->plan_of_n.find(n_plan);
        }
        const sconv_csr::Planned &p = planned->second;
        auto choice_for = [&](int n) -> const sconv_csr::Choice & { return choose_kernel(h, false, n, planned_us(h, n, p.us, p.phase_cg), p.plan.splits); };
        // batches of 1-4 share a tiling: sconv_forward_noalloc takes all of them once one has run, so their kernels are chosen
        // together and the LDS kernel's arrays go up as well
        if (N <= 4 && !h->conv_alt.choice_of_n.count(N))
            for (int n = 1; n <= 4; ++n) (void)choice_for(n);
        const sconv_csr::Choice &chosen = choice_for(N);
        if (chosen.kind != sconv_csr::kLds && is_flat_kernel(p.plan.kernel)) {
            *c = &chosen;
            if (N > 4) when = kPackLater;
        }
    }
    if (n_plan != h->planned_n || (when == kPackNow && h->flat && !is_packed(h->lds_flat))) return plan_lds(h, n_plan, when);
    return SCONV_OK;
}

// The per-row-stream kernel's tiles of 4 images and more are no match for the direct kernel on 1-3 images.
static bool runs_lds(const sconv_csr *h, int N)
{
    return h->has_lds && (h->flat || h->requested.kernel != 0 || N >= 4 || h->lds.t.p.nt < 4);
}

// The flat-stream kernel stages an unpadded strided layer straight from the input when its blocks hold whole phases; the other
// strided layers need a launch that writes the phase images.
static bool stages_phases(const sconv_csr *h) { return h->phased && h->flat && f_tiling(h).phase_cg > 0; }

// ws != nullptr: the caller forbids allocation.  Scratch then comes out of ws, and everything else the launch
// needs (the tiling for N, its packing, the device copies) must already exist: SCONV_ERR_PLAN otherwise.
static int forward_impl(sconv_csr *h, const float *in, float *out, int32_t N, const Epilogue &ep, void *hip_stream,
                        Workspace *ws)
{
    if (!h || !in || !out) return SCONV_ERR_NULL;
    if (N < 1) return SCONV_ERR_BATCH;
    const Geometry og = geometry(h->desc);
    const int64_t out_rows = (int64_t)N * h->desc.K, out_inner = (int64_t)og.OH * og.OW;
    if (ws) {
        const int n_plan = planned_batch(N);
        if (may_choose(h)) {
            // the other kernels' arrays are the same for every batch size: nothing has to be looked up or switched
            const auto planned = h->plan_of_n.find(n_plan);
            const auto known = h->conv_alt.choice_of_n.find(N);
            if (planned != h->plan_of_n.end() && known != h->conv_alt.choice_of_n.end() && known->second.kind != sconv_csr::kLds &&
                resident(h, h->conv_alt, known->second)) {
                // what this entry point takes does not depend on which kernel serves a call
                if (lds_scratch(h, N, planned->second) > ws->bytes) return SCONV_ERR_CAPACITY;
                return launch_choice(h, false, known->second, in, out, N, ep, hip_stream, ws);
            }
        }
        if (h->has_lds && free_choice(h) && n_plan != h->planned_n) {
            try {
                const int prc = plan_lds(h, n_plan, kResidentOnly);
                if (prc) return prc;
            } catch (const std::bad_alloc &) {
                return SCONV_ERR_NOMEM;
            }
        }
        if (!(h->has_lds && h->flat && h->lds_uploaded)) return SCONV_ERR_PLAN;
    } else {
        try {
            const sconv_csr::Choice *c;
            const int prc = decide(h, N, &c);
            if (prc) return prc;
            if (c && ready(h, false, N, *c)) {
                find_static_scratch();
                const int rc = N <= 4 ? upload_flat(h) : SCONV_OK;
                return rc ? rc : launch_choice(h, false, *c, in, out, N, ep, hip_stream);
            }
            if (c && h->flat) {
                const int rc = pack_now(h->kdesc, h->kc(), h->lds_flat);
                if (rc) return rc;
            }
        } catch (const std::bad_alloc &) {
            return SCONV_ERR_NOMEM;
        }
    }
    const bool use_lds = runs_lds(h, N), stage_phases = use_lds && stages_phases(h);
    int rc;
    if (use_lds && h->phased && !stage_phases) {
        // re-order the input into phase images (scratch owned by the handle, grown on demand)
        const size_t need = (size_t)N * h->kdesc.C * h->kdesc.H * h->kdesc.W * sizeof(float);
        float *phase;
        if (ws) {
            phase = static_cast<float *>(ws->take(need));
            if (!phase) return SCONV_ERR_CAPACITY;
        } else {
            rc = grow(&h->phase_buf, &h->phase_bytes, need, &h->hip_err);
            if (rc) return rc;
            phase = static_cast<float *>(h->phase_buf);
        }
        rc = launch_phase(h->desc, h->kdesc, in, phase, N, hip_stream, &h->hip_err);
        if (rc) return rc;
        in = phase;
    }
    if (use_lds && h->flat) {
        if (!h->lds_uploaded) {
            rc = upload_flat(h);
            if (rc) return rc;
            find_static_scratch();
        }
        const LdsTiling &ft = f_tiling(h);
        Lds2Layout lay = nchw_layout(h->kdesc, ft);
        if (stage_phases) {
            // the input side of the layout is the caller's tensor; the output side is the same for both forms
            const int64_t HW = (int64_t)h->desc.H * h->desc.W;
            lay.phase_stride = h->desc.stride;
            lay.src_w = h->desc.W;
            lay.in_img = h->desc.C * HW; lay.in_tile = 4 * lay.in_img; lay.in_ch = HW; lay.in_pos = 1;
            lay.in_rec_fixed = 0; lay.in_rec_img = lay.in_img * 4; lay.in_rec_tile = 0;
        }
        return run_flat(h, h->kdesc, ft, h->dev_lds, lay, in, out, N, out_rows, out_inner, ep, hip_stream, ws);
    }
    if (use_lds) {
        if (!h->lds_uploaded) {
            rc = upload(h->lds.pairs.data(), h->lds.pairs.size() * 8, &h->dev_lds.pairs, &h->hip_err);
            if (!rc) rc = upload(h->lds.seg_ptr.data(), h->lds.seg_ptr.size() * 4, &h->dev_lds.seg_ptr, &h->hip_err);
            if (!rc) rc = upload(h->lds.row_of.data(), h->lds.row_of.size() * 4, &h->dev_lds.row_of, &h->hip_err);
            if (rc) return rc;
            h->lds_uploaded = true;
        }
        rc = launch_lds(h->kdesc, h->lds.t, h->dev_lds, in, out, N, hip_stream, &h->hip_err);
        return rc ? rc : launch_epilogue(out, out_rows, out_inner, h->desc.K, ep, hip_stream, &h->hip_err);
    }
    rc = upload_direct(h);
    if (rc) return rc;
    rc = launch_direct(h->desc, h->dev_direct, in, out, N, hip_stream, &h->hip_err);
    return rc ? rc : launch_epilogue(out, out_rows, out_inner, h->desc.K, ep, hip_stream, &h->hip_err);
}

static sconv_route route_of_choice(const sconv_desc &d, bool fc, const sconv_csr::Choice &c)
{
    if (c.kind == sconv_csr::kMfma) return {SCONV_KERNEL_MFMA, c.mfma.splits > 1 ? 2 : 1, c.mfma.mt, c.mfma.nt, c.mfma.splits};
    if (c.kind == sconv_csr::kFlatMc) return {SCONV_KERNEL_FLAT_MC, c.mc.splits > 1 ? 2 : 1, c.mc.mt, c.mc.nt, c.mc.splits};
    const int kernel = fc ? SCONV_KERNEL_FC_GATHER : gather4_fits(d) ? SCONV_KERNEL_GATHER4 : SCONV_KERNEL_GATHER;
    return {kernel, 1, c.gather.t, 1, c.gather.split};
}

static sconv_route route_of_flat(const sconv_plan &p, int launches) { return {p.kernel, launches + (p.splits > 1), p.t, 1, p.splits}; }

extern "C" int sconv_route_of(sconv_csr *h, int32_t N, sconv_route *route)
{
    if (!h || !route) return SCONV_ERR_NULL;
    if (N < 1) return SCONV_ERR_BATCH;
    try {
        const sconv_csr::Choice *c;
        const int rc = decide(h, N, &c);
        if (rc) return rc;
        if (c)
            *route = route_of_choice(h->desc, false, *c);
        else if (!runs_lds(h, N))
            *route = {SCONV_KERNEL_DIRECT, 1, 0, 0, 1};
        else if (h->flat)
            *route = route_of_flat(f_tiling(h).p, h->phased && !stages_phases(h) ? 2 : 1);
        else
            *route = {SCONV_KERNEL_ROWS, h->phased ? 2 : 1, h->lds.t.p.t, 1, 1};
    } catch (const std::bad_alloc &) {
        return SCONV_ERR_NOMEM;
    }
    return SCONV_OK;
}

extern "C" int sconv_forward_noalloc(sconv_csr *h, const float *in, float *out, int32_t N, void *hip_stream)
{
    if (!h) return SCONV_ERR_NULL;
    Workspace ws;
    void *base = nullptr;
    const int rc = static_scratch(&base, &ws.bytes, &h->hip_err);
    if (rc) return rc;
    ws.base = static_cast<char *>(base);
    return forward_impl(h, in, out, N, Epilogue(), hip_stream, &ws);
}

// ---- fully connected layers: out_t[K][N] = W[K][C] (CSR) x in_t[C][N] -------------------------------
//
// With the activations feature-major, four consecutive images of one feature are exactly one LDS cell of
// the flat-stream kernel and a feature's row is a channel plane: the product is the 1x1 convolution of a
// C-channel "image" of N/4 positions x 4 images, and the kernel runs it unchanged through other strides.

static bool is_fc(const sconv_desc &d)
{
    return d.H == 1 && d.W == 1 && d.R == 1 && d.S == 1 && d.stride == 1 && d.pad == 0 && d.groups == 1;
}

static void release_fc(sconv_csr *h)
{
    release(h->fc_dev.pairs);
    release(h->fc_dev.seg_ptr);
    release(h->fc_dev.row_of);
    release(h->fc_dev.store_tbl);
    h->fc_dev = DeviceLds();
    h->fc_uploaded = false;
}

// The layer as the flat-stream kernel sees it for a batch of N: `tiles` tiles of N / tiles images, f
// consecutive features forming one channel of f rows (a filter of f x 1 taps, one output row): the same
// arithmetic, but a channel plane is f times larger, so that every wave of a workgroup has a part of it
// to stage when the batch alone gives a plane of only a few hundred floats.
static int fc_mapping(const sconv_csr *h, int N, sconv_desc &kd, int &tiles)
{
    if (!is_fc(h->desc)) return SCONV_ERR_DESC;
    if (N < 4 || N % 4) return SCONV_ERR_BATCH;
    // one wave covers at most 4 x 256 images; larger batches are cut into equal tiles
    tiles = (N + 1023) / 1024;
    if (N % (4 * tiles)) return SCONV_ERR_BATCH;
    const int nc = N / tiles;
    int f = 1;
    if (tiles == 1)
        for (int c : {16, 8, 4, 2})
            if (h->desc.C % c == 0 && c * nc <= 1024) {
                f = c;
                break;
            }
    kd = h->desc;
    kd.C = h->desc.C / f;
    kd.H = f;
    kd.R = f;
    kd.W = nc / 4;
    return SCONV_OK;
}

// What the tiling search is asked for: the fields of the plan the handle was created with are honoured
// where they apply to this mapping.
static sconv_plan fc_request(const sconv_csr *h)
{
    sconv_plan req = h->requested;
    req.kernel = (req.kernel == 3 || req.kernel == 4) ? req.kernel : 0; // tiles of four images: a flat-stream variant either way
    req.nt = 4;
    req.band = 0;
    req.strip = 0;
    return req;
}

// The layer's CSR in the wide image's terms: feature c = row c.
static Canonical fc_canonical(const sconv_csr *h, const sconv_desc &kd)
{
    Canonical kc = h->canon;
    for (int32_t &off : kc.off) off *= kd.W;
    return kc;
}

static int pack_fc(sconv_csr *h)
{
    return is_packed(h->fc_flat) ? SCONV_OK : pack_now(h->fc_desc, fc_canonical(h, h->fc_desc), h->fc_flat);
}

// Plan for a batch of N, and pack unless `later` (then pack_fc does).  force: a complete tiling to use (sconv_fc_tune's
// candidates); otherwise the one tuned for N if there is one, otherwise the cost model's choice.
static int plan_fc(sconv_csr *h, int N, const sconv_csr::Planned *force = nullptr, bool later = false)
{
    sconv_desc kd;
    int tiles;
    int rc = fc_mapping(h, N, kd, tiles);
    if (rc) return rc;
    if (!force) {
        auto tuned = h->fc_plan_of_n.find(N);
        if (tuned != h->fc_plan_of_n.end()) force = &tuned->second;
    }
    if (N == h->fc_n && (!force || same_plan(force->plan, h->fc_flat.t.p))) return later ? SCONV_OK : pack_fc(h);
    if (h->fc_n > 0) { // set the current packing aside; one for this batch size may be waiting there
        StashedPacking old;
        old.flat = true;
        old.lds_flat = std::move(h->fc_flat);
        old.dev = h->fc_dev;
        old.uploaded = h->fc_uploaded;
        old.fc_n = h->fc_n;
        old.fc_tiles = h->fc_tiles;
        old.fc_desc = h->fc_desc;
        h->fc_stash.push_back(std::move(old));
        h->fc_dev = DeviceLds();
        h->fc_uploaded = false;
        h->fc_n = 0;
        while (h->fc_stash.size() > h->stash_cap) {
            release_arrays(h->fc_stash.front().dev);
            h->fc_stash.erase(h->fc_stash.begin());
        }
    }
    for (size_t i = 0; i < h->fc_stash.size(); ++i) {
        StashedPacking &sp = h->fc_stash[i];
        if (sp.fc_n != N || (force && !same_plan(force->plan, sp.lds_flat.t.p))) continue;
        h->fc_flat = std::move(sp.lds_flat);
        h->fc_dev = sp.dev;
        h->fc_uploaded = sp.uploaded;
        h->fc_tiles = sp.fc_tiles;
        h->fc_desc = sp.fc_desc;
        h->fc_n = N;
        h->fc_stash.erase(h->fc_stash.begin() + (long)i);
        return later ? SCONV_OK : pack_fc(h);
    }
    LdsTiling t;
    rc = make_lds_tiling(kd, force ? force->plan : fc_request(h), 4 * tiles, avg_row_nnz(h), t, 0, true);
    if (rc) return rc;
    if (force) t.us = force->us; // (a complete tiling is not searched for, so not priced either)
    t.out_pos = 4; // the four images of a cell are consecutive in the output row
    h->fc_flat = PackedFlat();
    h->fc_flat.t = t;
    h->fc_desc = kd;
    h->fc_tiles = tiles;
    rc = later ? SCONV_OK : pack_fc(h);
    if (!rc) h->fc_n = N;
    return rc;
}

// The same decision for the fully connected entry point, against the tiling just planned.
static const sconv_csr::Choice &choose_fc_kernel(sconv_csr *h, int N)
{
    if (free_choice(h) && h->requested.kernel == 0) return choose_kernel(h, true, N, h->fc_flat.t.us, h->fc_flat.t.p.splits);
    static const sconv_csr::Choice lds = {sconv_csr::kLds, {0, 0, 0.0, 0.0}, {}, {}, false};
    return lds;
}

extern "C" int sconv_fc_plan(sconv_csr *h, int32_t N, sconv_plan *plan)
{
    if (!h || !plan) return SCONV_ERR_NULL;
    try {
        const int rc = plan_fc(h, N);
        if (rc) return rc;
    } catch (const std::bad_alloc &) {
        return SCONV_ERR_NOMEM;
    }
    *plan = h->fc_flat.t.p;
    return SCONV_OK;
}

extern "C" int sconv_fc_route_of(sconv_csr *h, int32_t N, sconv_route *route)
{
    if (!h || !route) return SCONV_ERR_NULL;
    try {
        const int rc = plan_fc(h, N, nullptr, true);
        if (rc) return rc;
        const sconv_csr::Choice &c = choose_fc_kernel(h, N);
        *route = c.kind != sconv_csr::kLds ? route_of_choice(h->desc, true, c) : route_of_flat(h->fc_flat.t.p, 1);
    } catch (const std::bad_alloc &) {
        return SCONV_ERR_NOMEM;
    }
    return SCONV_OK;
}

extern "C" int sconv_fc_forward(sconv_csr *h, const float *in_t, float *out_t, int32_t N, const float *bias, int32_t relu,
                                void *hip_stream)
{
    if (!h || !in_t || !out_t) return SCONV_ERR_NULL;
    if (N < 1) return SCONV_ERR_BATCH;
    Epilogue ep;
    ep.bias = bias;
    ep.relu = relu != 0;
    int rc;
    try {
        rc = plan_fc(h, N, nullptr, true);
        if (rc) return rc;
        const sconv_csr::Choice &c = choose_fc_kernel(h, N);
        if (c.kind != sconv_csr::kLds && ready(h, true, N, c)) return launch_choice(h, true, c, in_t, out_t, N, ep, hip_stream);
        rc = pack_fc(h);
        if (rc) return rc;
    } catch (const std::bad_alloc &) {
        return SCONV_ERR_NOMEM;
    }
    if (!h->fc_uploaded) {
        const PackedFlat &f = h->fc_flat;
        rc = upload(f.pairs.data(), f.pairs.size() * 8, &h->fc_dev.pairs, &h->hip_err);
        if (!rc) rc = upload(f.seg.data(), f.seg.size() * 4, &h->fc_dev.seg_ptr, &h->hip_err);
        if (!rc) rc = upload(f.row_of.data(), f.row_of.size() * 4, &h->fc_dev.row_of, &h->hip_err);
        if (!rc) rc = upload(f.store_tbl.data(), f.store_tbl.size() * 4, &h->fc_dev.store_tbl, &h->hip_err);
        if (rc) {
            release_fc(h);
            return rc;
        }
        h->fc_uploaded = true;
    }
    const LdsTiling &t = h->fc_flat.t;
    const int64_t C = h->desc.C, K = h->desc.K, nc = N / h->fc_tiles;
    Lds2Layout lay;
    lay.in_tile = nc; lay.in_img = 1; lay.in_ch = (int64_t)h->fc_desc.H * N; lay.in_pos = 4;
    lay.in_rec_fixed = C * N * 4; lay.in_rec_img = 0; lay.in_rec_tile = nc * 4;
    lay.out_tile = nc; lay.out_band = 0; lay.out_row = N; lay.out_img = 1; lay.out_pos = 4;
    return run_flat(h, h->fc_desc, t, h->fc_dev, lay, in_t, out_t, 4 * h->fc_tiles, K, N, ep, hip_stream);
}

// ---- measured choice of the tiling ----------------------------------------------------------------------

// Times run() after install(i) for candidates 0 .. n-1 and returns the index of the fastest in *best
// (-1 if none could be installed and run).  A candidate that cannot be packed or launched is skipped; candidate
// `own` is the one an untuned call uses.
// All candidates are packed and uploaded first and stay in the handle's stash, so that the timed part only
// switches between them: the GPU's clocks drop while the host packs, and a candidate timed right after
// that would look 10-15 % slower than one timed later.
template <class Install, class Run>
static int time_candidates(sconv_csr *h, size_t n, size_t own, Install install, Run run, void *stream, int *best)
{
    *best = -1;
    std::vector<size_t> ok;
    for (size_t i = 0; i < n; ++i)
        if (install(i) == SCONV_OK && run() == SCONV_OK) ok.push_back(i);
    if (ok.empty()) return SCONV_OK;
    StreamTimer timer;
    int rc = timer_create(timer, &h->hip_err);
    if (rc) return rc;
    // `n` runs between two events, in milliseconds per run
    auto timed = [&](int n, float *ms) {
        int r = timer_start(timer, stream, &h->hip_err);
        for (int k = 0; k < n && !r; ++k) r = run();
        if (!r) r = timer_stop_ms(timer, stream, ms, &h->hip_err);
        *ms /= (float)n;
        return r;
    };
    // warm-up, about 30 ms of the first candidate
    float ms = 0, spent = 0;
    rc = install(ok[0]);
    for (int k = 0; k < 200 && !rc && spent < 30.0f; ++k) {
        rc = timed(4, &ms);
        spent += 4 * ms;
    }
    // three rounds over the candidates, about 2 ms each; a candidate's time is its fastest round
    std::vector<float> t(ok.size(), std::numeric_limits<float>::max());
    for (int round = 0; round < 3 && !rc; ++round)
        for (size_t j = 0; j < ok.size() && !rc; ++j) {
            rc = install(ok[j]);
            if (!rc) rc = timed(1, &ms);
            if (rc) break;
            const int reps = std::max(3, std::min(40, (int)(2.0f / std::max(ms, 0.01f))));
            rc = timed(reps, &ms);
            if (!rc) t[j] = std::min(t[j], ms);
        }
    timer_destroy(timer);
    if (rc) return rc;
    size_t arg = 0;
    for (size_t j = 1; j < ok.size(); ++j)
        if (t[j] < t[arg]) arg = j;
    // the timings repeat to 1-2 %: the cost model's own choice stands unless another is clearly faster
    for (size_t j = 0; j < ok.size(); ++j)
        if (ok[j] == own && t[arg] > 0.985f * t[j]) arg = j;
    *best = (int)ok[arg];
    return SCONV_OK;
}

// The stash holds every candidate while they are timed; afterwards the oldest go.
struct StashRoom {
    sconv_csr *h;
    StashRoom(sconv_csr *handle, size_t n) : h(handle) { h->stash_cap = std::max(kStashed, n); }
    ~StashRoom()
    {
        h->stash_cap = kStashed;
        while (h->stash.size() > kStashed) {
            release_arrays(h->stash.front().dev);
            h->stash.erase(h->stash.begin());
        }
        while (h->fc_stash.size() > kStashed) {
            release_arrays(h->fc_stash.front().dev);
            h->fc_stash.erase(h->fc_stash.begin());
        }
    }
};

// The kernels besides the flat-stream one that can take a call.
static std::vector<sconv_csr::Kind> other_kernels(const sconv_csr::Choice &c)
{
    std::vector<sconv_csr::Kind> k;
    if (c.gather.t > 0) k.push_back(sconv_csr::kGather);
    if (c.mfma.mt > 0) k.push_back(sconv_csr::kMfma);
    if (c.mc.mt > 0) k.push_back(sconv_csr::kFlatMc);
    return k;
}

static int clamp_plans(int max_plans) { return max_plans < 1 ? 8 : std::min(max_plans, 32); }

extern "C" int sconv_rank_plans(const sconv_csr *h, int32_t N, int32_t max_plans, sconv_plan *plans, int32_t *count)
{
    if (!h || !plans || !count) return SCONV_ERR_NULL;
    *count = 0;
    if (N < 1) return SCONV_ERR_BATCH;
    if (!h->has_lds) return SCONV_ERR_PLAN;
    try {
        const double avg = h->kdesc.K ? (double)h->canon.val.size() / h->kdesc.K : 0.0;
        std::vector<LdsTiling> cands;
        const int rc = rank_lds_tilings(h->kdesc, h->requested, N < 4 ? 4 : N, avg, clamp_plans(max_plans), cands, h->phase_cg());
        if (rc) return rc;
        for (const LdsTiling &t : cands) plans[(*count)++] = t.p;
    } catch (const std::bad_alloc &) {
        return SCONV_ERR_NOMEM;
    }
    return SCONV_OK;
}

extern "C" int sconv_tune(sconv_csr *h, const float *in, float *out, int32_t N, int32_t max_plans, void *hip_stream)
{
    if (!h || !in || !out) return SCONV_ERR_NULL;
    if (N < 1) return SCONV_ERR_BATCH;
    if (!h->has_lds || !free_choice(h)) return SCONV_ERR_PLAN;
    const int n_plan = N < 4 ? 4 : N;
    const Epilogue none;
    try {
        const double avg = h->kdesc.K ? (double)h->canon.val.size() / h->kdesc.K : 0.0;
        std::vector<LdsTiling> cands;
        int rc = rank_lds_tilings(h->kdesc, h->requested, n_plan, avg, clamp_plans(max_plans), cands, h->phase_cg());
        if (rc) return rc;
        int best = -1;
        StashRoom room(h, cands.size());
        // the other kernels are further candidates where they can run (and the untuned choice where the models pick one)
        h->conv_alt.choice_of_n.erase(N);
        const size_t n_lds = cands.size();
        sconv_csr::Choice own = {sconv_csr::kLds, {0, 0, 0.0, 0.0}, {}, {}, false};
        if (h->requested.kernel == 0 && h->flat) own = choose_kernel(h, false, N, planned_us(h, N, cands[0].us, cands[0].phase_cg), cands[0].p.splits);
        const std::vector<sconv_csr::Kind> others = other_kernels(own);
        auto choice = [&](size_t i) {
            sconv_csr::Choice c = own;
            c.kind = i < n_lds ? sconv_csr::kLds : others[i - n_lds];
            c.tuned = true;
            return c;
        };
        size_t own_index = 0;
        for (size_t i = 0; i < others.size(); ++i)
            if (own.kind == others[i]) own_index = n_lds + i;
        auto install = [&](size_t i) {
            h->conv_alt.choice_of_n[N] = choice(i);
            const LdsTiling &c = cands[i < n_lds ? i : 0];
            h->plan_of_n[n_plan] = {c.p, c.us, c.phase_cg, true};
            return plan_lds(h, n_plan);
        };
        rc = time_candidates(h, n_lds + others.size(), own_index, install,
                             [&]() { return forward_impl(h, in, out, N, none, hip_stream); }, hip_stream, &best);
        // the fastest, or the cost models' choice if nothing could be timed
        const size_t winner = best < 0 ? own_index : (size_t)best;
        h->conv_alt.choice_of_n[N] = choice(winner);
        const LdsTiling &c = cands[winner < n_lds ? winner : 0];
        h->plan_of_n[n_plan] = {c.p, c.us, c.phase_cg, true};
        const int prc = plan_lds(h, n_plan);
        if (rc) return rc;
        if (prc) return prc;
    } catch (const std::bad_alloc &) {
        return SCONV_ERR_NOMEM;
    }
    return forward_impl(h, in, out, N, none, hip_stream);
}

extern "C" int sconv_fc_tune(sconv_csr *h, const float *in_t, float *out_t, int32_t N, int32_t max_plans, void *hip_stream)
{
    if (!h || !in_t || !out_t) return SCONV_ERR_NULL;
    if (N < 1) return SCONV_ERR_BATCH;
    try {
        sconv_desc kd;
        int tiles;
        int rc = fc_mapping(h, N, kd, tiles);
        if (rc) return rc;
        const double avg = kd.K ? (double)h->canon.val.size() / kd.K : 0.0;
        std::vector<LdsTiling> cands;
        rc = rank_lds_tilings(kd, fc_request(h), 4 * tiles, avg, clamp_plans(max_plans), cands, 0, true);
        if (rc) return rc;
        int best = -1;
        StashRoom room(h, cands.size());
        h->fc_plan_of_n.erase(N);
        h->fc_alt.choice_of_n.erase(N);
        const size_t n_lds = cands.size();
        auto planned = [&](size_t i) {
            const LdsTiling &c = cands[i < n_lds ? i : 0];
            return sconv_csr::Planned{c.p, c.us, c.phase_cg, true};
        };
        const sconv_csr::Planned first = planned(0);
        rc = plan_fc(h, N, &first);
        if (rc) return rc;
        const sconv_csr::Choice own = choose_fc_kernel(h, N);
        const std::vector<sconv_csr::Kind> others = other_kernels(own);
        auto choice = [&](size_t i) {
            sconv_csr::Choice c = own;
            c.kind = i < n_lds ? sconv_csr::kLds : others[i - n_lds];
            c.tuned = true;
            return c;
        };
        size_t own_index = 0;
        for (size_t i = 0; i < others.size(); ++i)
            if (own.kind == others[i]) own_index = n_lds + i;
        rc = time_candidates(
            h, n_lds + others.size(), own_index,
            [&](size_t i) {
                h->fc_alt.choice_of_n[N] = choice(i);
                const sconv_csr::Planned c = planned(i);
                return plan_fc(h, N, &c);
            },
            [&]() { return sconv_fc_forward(h, in_t, out_t, N, nullptr, 0, hip_stream); }, hip_stream, &best);
        // the fastest, or the cost models' choice if nothing could be timed
        const size_t winner = best < 0 ? own_index : (size_t)best;
        h->fc_alt.choice_of_n[N] = choice(winner);
        h->fc_plan_of_n[N] = planned(winner);
        const int prc = plan_fc(h, N); // while the candidates' packings are still at hand
        if (rc) return rc;
        if (prc) return prc;
    } catch (const std::bad_alloc &) {
        return SCONV_ERR_NOMEM;
    }
    return sconv_fc_forward(h, in_t, out_t, N, nullptr, 0, hip_stream);
}

extern "C" int sconv_last_hip_error(const sconv_csr *h) { return h ? h->hip_err : 0; }

extern "C" void sconv_destroy_csr(sconv_csr *h)
{
    if (!h) return;
    release(h->dev_lds.pairs);
    release(h->dev_lds.seg_ptr);
    release(h->dev_lds.row_of);
    release(h->dev_lds.store_tbl);
    release(h->phase_buf);
    release(h->part_buf);
    release_fc(h);
    for (auto &sp : h->stash) release_arrays(sp.dev);
    for (auto &sp : h->fc_stash) release_arrays(sp.dev);
    release(h->dev_direct.rowptr);
    release(h->dev_direct.trip);
    for (sconv_csr::Alternatives *alt : {&h->conv_alt, &h->fc_alt}) {
        release_gather(alt->gather);
        release_mfma(alt->mfma);
    }
    release_arrays(h->flat_mc.dev);
    delete h;
}

extern "C" const char *sconv_strerror(int status)
{
    switch (status) {
    case SCONV_OK: return "ok";
    case SCONV_ERR_NULL: return "a required pointer is NULL";
    case SCONV_ERR_DESC: return "bad layer descriptor";
    case SCONV_ERR_CSR: return "malformed CSR arrays";
    case SCONV_ERR_BATCH: return "batch size below 1, or not one the fully connected path takes (a multiple of 4 per tile)";
    case SCONV_ERR_CAPACITY: return "output buffer too small";
    case SCONV_ERR_PLAN: return "tiling not runnable for this layer";
    case SCONV_ERR_HIP: return "HIP call failed";
    case SCONV_ERR_NOMEM: return "out of host memory";
    case SCONV_ERR_RANGE: return "sizes exceed 32-bit offsets";
    default: return "unknown status";
    }
}

// ------------------------------------------------------------------------------------------------
// Section 2.2: t_dense = C/F, t_sparse_compute = alpha*x*C/F, t_sparse_bw = (S_A + beta*x*S_W)/B,
// speedup = t_dense / max(t_sparse_compute, t_sparse_bw).

extern "C" void sconv_machine_gfx950(sconv_machine *m)
{
    if (!m) return;
    // Achievable rates measured on one MI355X (see the benchmark report); not data-sheet peaks.
    m->dense_flops = 100e12;        // fp32 dense convolution / SGEMM proxy
    m->hbm_bytes_per_s = 4.9e12;    // device copy kernel (read + write), 1 GiB
    m->alpha = 0.0;                 // derive from the ceilings below
    m->beta = 2.0;
    m->fma_flops = 73.5e12;         // v_fma_f32, 256 CUs x 60 lanes-FMA/clk x 2.4 GHz x 2
    m->lds_bytes_per_s = 148e12;    // aligned ds_read_b128, 242 B/clk/CU
    m->lds_bytes_per_fma = 4.0;
    m->lane_efficiency = 0.73;      // 0.9 (lanes that are outputs) x 0.8 (issue slots left after address
                                    // arithmetic, LDS waits and barriers): CALIBRATED to the measured x = 1
                                    // plateau of 53-55 TFLOP/s, as the paper takes alpha from its measured plateau
    m->t_fixed = 11.4e-6;           // intercept of time against nonzeros on conv3's shape at batch 256
}

static int predict(const sconv_desc *desc, int32_t N, double density, const sconv_csr *h, const sconv_machine *m,
                   bool lowered, sconv_prediction *out);

extern "C" int sconv_model_predict(const sconv_desc *desc, int32_t N, double density, const sconv_csr *h,
                                   const sconv_machine *m, sconv_prediction *out)
{
    return predict(desc, N, density, h, m, false, out);
}

extern "C" int sconv_model_predict_lowered(const sconv_desc *desc, int32_t N, double density, const sconv_csr *h,
                                           const sconv_machine *m, sconv_prediction *out)
{
    return predict(desc, N, density, h, m, true, out);
}

static int predict(const sconv_desc *desc, int32_t N, double density, const sconv_csr *h, const sconv_machine *m,
                   bool lowered, sconv_prediction *out)
{
    if (!desc || !out) return SCONV_ERR_NULL;
    int rc = validate_desc(*desc);
    if (rc) return rc;
    if (N < 1) return SCONV_ERR_BATCH;
    sconv_machine def;
    if (!m) {
        sconv_machine_gfx950(&def);
        m = &def;
    }
    const Geometry g = geometry(*desc);
    const double cols = (double)g.Cg * desc->R * desc->S;
    double x = density;
    if (h) x = (double)h->canon.val.size() / ((double)desc->K * cols);
    if (!(x >= 0.0) || !(m->dense_flops > 0) || !(m->hbm_bytes_per_s > 0)) return SCONV_ERR_DESC;
    double alpha = m->alpha;
    if (!(alpha > 0)) {
        const double lds_flops = 2.0 * m->lds_bytes_per_s / m->lds_bytes_per_fma;
        const double f_sparse = m->lane_efficiency * std::fmin(m->fma_flops, lds_flops);
        if (!(f_sparse > 0)) return SCONV_ERR_DESC;
        alpha = m->dense_flops / f_sparse;
    }
    sconv_prediction p;
    p.flops_dense = 2.0 * desc->K * cols * g.OH * g.OW * N;
    // direct: every input element once; lowered: the (C*R*S) x (OH*OW) matrix the lowering writes out
    const double in_elems = lowered ? (double)desc->C * desc->R * desc->S * g.OH * g.OW : (double)desc->C * desc->H * desc->W;
    p.bytes_act = 4.0 * N * (in_elems + (double)desc->K * g.OH * g.OW);
    p.bytes_w = 4.0 * desc->K * cols;
    p.density = x;
    p.alpha = alpha;
    p.t_dense = p.flops_dense / m->dense_flops;
    p.t_sparse_compute = alpha * x * p.flops_dense / m->dense_flops;
    p.t_sparse_bw = (p.bytes_act + m->beta * x * p.bytes_w) / m->hbm_bytes_per_s;
    p.t_sparse = std::fmax(p.t_sparse_compute, p.t_sparse_bw) + (m->t_fixed > 0 ? m->t_fixed : 0.0);
    p.speedup = p.t_dense / p.t_sparse;
    p.effective_flops = p.flops_dense / p.t_sparse;
    p.actual_flops = x * p.flops_dense / p.t_sparse;
    const double denom = alpha * p.flops_dense / m->dense_flops - m->beta * p.bytes_w / m->hbm_bytes_per_s;
    p.x_upper = denom > 0 ? (p.bytes_act / m->hbm_bytes_per_s) / denom : std::numeric_limits<double>::infinity();
    p.x_lower = 1.0 / alpha;
    p.bandwidth_bound = p.t_sparse_bw > p.t_sparse_compute ? 1 : 0;
    *out = p;
    return SCONV_OK;
}

// Section 2.3's algorithm, one layer, one decision: exclude layers without a useful sparsity range at the
// start; stop pruning a layer once its sparsity reaches the upper bound of the range (density <= x_upper);
// give up on a layer whose sparsity has stabilised at or below the lower bound (density >= x_lower) and
// restore its dense weights; otherwise keep pruning.
extern "C" int sconv_gsl_decide(const sconv_desc *desc, int32_t N, double density, int32_t stabilized,
                                const sconv_machine *m, int32_t *action, sconv_prediction *pred)
{
    if (!action) return SCONV_ERR_NULL;
    if (!(density > 0.0) || density > 1.0) return SCONV_ERR_DESC;
    sconv_prediction p;
    const int rc = sconv_model_predict(desc, N, density, nullptr, m, &p);
    if (rc) return rc;
    if (pred) *pred = p;
    if (!(p.x_upper < p.x_lower))
        *action = SCONV_GSL_EXCLUDE;
    else if (density <= p.x_upper)
        *action = SCONV_GSL_STOP;
    else if (stabilized && density >= p.x_lower)
        *action = SCONV_GSL_RESTORE_DENSE;
    else
        *action = SCONV_GSL_PRUNE;
    return SCONV_OK;
}
