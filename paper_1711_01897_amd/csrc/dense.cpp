// P1 and DP1 blocks by triangle pairs (the dense weak-form assembly of
// Section 3): every regular triangle pair of star(rows) x star(cols) is
// integrated once into its 3 x 3 local matrix on the device, then each entry
// adds its pairs' local values in a fixed order (entries.hip: k_local_*,
// k_gather_pairs).  Device-tensor requests large enough take it
// (pairs_pay); bem_eval_dense is the host form: rows go in panels whose local
// matrices fit a device budget; the panels run on a compute stream while a
// copy stream moves the previous panel's entries to pinned host memory and a few
// threads copy the one before into `out`, so assembly and transfer overlap
// (Section 3's chunked assembly with overlapped transfers).
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <memory>
#include <mutex>

#include "bem_internal.hpp"
#include "host_copy.hpp"

namespace bem {

hipError_t launch_pair_local(int op, bool fp32, bool ltrial, const bem_mesh &m, const int32_t *ftri, int nf,
                             const int32_t *ltri, int nl, void *Lr, void *Li, double k, hipStream_t s);
hipError_t launch_pair_gather(bool fp32, bool cplx, const void *Lr, const void *Li, int nl, const int32_t *fptr,
                              const int32_t *fsrc, const int32_t *fpos, int nfd, const int32_t *lptr,
                              const int32_t *lsrc, const int32_t *lpos, int nld, void *out, int64_t sf, int64_t sl,
                              hipStream_t s);

namespace {

// Per-thread marks of triangles: index within the open panel.
struct PairScratch {
    std::vector<uint32_t> stamp;
    std::vector<int32_t> index;
    uint32_t gen = 0;
    void open(int64_t nt)
    {
        if ((int64_t)stamp.size() < nt) {
            stamp.assign((size_t)nt, 0);
            index.resize((size_t)nt);
            gen = 0;
        }
        if (++gen == 0) {
            std::fill(stamp.begin(), stamp.end(), 0);
            gen = 1;
        }
    }
};
thread_local PairScratch g_pair;

void star_range(const bem_mesh &m, int space, int32_t d, int64_t &b, int64_t &e)
{
    if (space == BEM_P1) {
        b = m.star_ptr[d];
        e = m.star_ptr[d + 1];
    } else {
        b = m.dp1_star[d];
        e = b + 1;
    }
}

// Cuts a side into panels of at most most_tri distinct triangles (one dof's
// star at least) and most_dof dofs.
void cut_side(const bem_mesh &m, int space, const int32_t *dofs, int64_t n, int64_t most_tri, int64_t most_dof,
              std::vector<int32_t> &ints, std::vector<PairPanel> &out)
{
    std::vector<int32_t> order, tri, ptr, src;
    morton_order(m, space, dofs, n, order);
    PairScratch &sc = g_pair;
    int64_t i = 0;
    while (i < n) {
        sc.open(m.nt);
        tri.clear();
        src.clear();
        ptr.assign(1, 0);
        const int64_t first = i;
        for (; i < n; ++i) {
            int64_t b, e, fresh = 0;
            star_range(m, space, dofs[order[i]], b, e);
            for (int64_t s = b; s < e; ++s) fresh += sc.stamp[m.star[s] >> 2] != sc.gen;
            if (i > first && ((int64_t)tri.size() + fresh > most_tri || i - first >= most_dof)) break;
            for (int64_t s = b; s < e; ++s) {
                const int32_t t = m.star[s] >> 2;
                if (sc.stamp[t] != sc.gen) {
                    sc.stamp[t] = sc.gen;
                    sc.index[t] = (int32_t)tri.size();
                    tri.push_back(t);
                }
                src.push_back((sc.index[t] << 2) | (m.star[s] & 3));
            }
            ptr.push_back((int32_t)src.size());
        }
        PairPanel P;
        P.ntri = (int32_t)tri.size();
        P.ndof = (int32_t)(i - first);
        auto put = [&](auto b, auto e) {
            const size_t at = ints.size();
            ints.insert(ints.end(), b, e);
            return at;
        };
        P.tri = put(tri.begin(), tri.end());
        P.ptr = put(ptr.begin(), ptr.end());
        P.src = put(src.begin(), src.end());
        P.pos = put(order.begin() + first, order.begin() + i);
        out.push_back(P);
    }
}

// Star entries and distinct triangles of a dof list.
void count_side(const bem_mesh &m, int space, const int32_t *dofs, int64_t n, int64_t &stars, int64_t &distinct)
{
    PairScratch &sc = g_pair;
    sc.open(m.nt);
    stars = distinct = 0;
    for (int64_t i = 0; i < n; ++i) {
        int64_t b, e;
        star_range(m, space, dofs[i], b, e);
        stars += e - b;
        for (int64_t s = b; s < e; ++s) {
            const int32_t t = m.star[s] >> 2;
            distinct += sc.stamp[t] != sc.gen;
            sc.stamp[t] = sc.gen;
        }
    }
}

// Triangles a panel takes at most, of `pairs` local matrices the workspace holds.
// Lane panels leave room for at least 64 fixed-side triangles (or the largest
// star); 262,144 of those: the launch grid's second dimension at four or more a
// workgroup.
struct PanelCut {
    int64_t pairs, lanes;
    int64_t fixed(int64_t nl) const { return std::min<int64_t>(std::max<int64_t>(1, pairs / nl), 65535 * 4); }
};

PanelCut panel_cut(const bem_mesh &m, size_t pairs)
{
    return {(int64_t)pairs, std::max<int64_t>(256, (int64_t)pairs / std::max<int64_t>(64, m.max_star))};
}

size_t pair_bytes(int op, int prec) { return 9 * (prec == BEM_FP32 ? 4 : 8) * (size_t)(is_complex_op(op) ? 2 : 1); }

}  // namespace

void plan_pairs(const bem_mesh &m, int space, int op, int prec, bool ltrial, const int32_t *fix, int64_t nfix,
                const int32_t *lane, int64_t nlane, size_t budget, PairPlan &P, bool entries_panelled)
{
    P.ints.clear();
    P.fix.clear();
    P.lane.clear();
    P.op = op;
    P.prec = prec;
    P.ltrial = ltrial;
    const size_t per = pair_bytes(op, prec);
    const PanelCut cut = panel_cut(m, budget / per);
    cut_side(m, space, lane, nlane, cut.lanes, nlane, P.ints, P.lane);
    int64_t nl = 1;
    for (const PairPanel &l : P.lane) nl = std::max<int64_t>(nl, l.ntri);
    // As many dofs as the gather's launch grid takes at four rows a workgroup; where a
    // panel's entries are held panel by panel, about as many as its triangles have
    // on a closed mesh (repeated dofs add rows but no triangles)
    const int64_t rows = entries_panelled ? std::min<int64_t>(65535, cut.fixed(nl) / 2 + 64) : 65535 * 4;
    cut_side(m, space, fix, nfix, cut.fixed(nl), rows, P.ints, P.fix);
    int64_t nf = 0;
    P.pairs = 0;
    for (const PairPanel &f : P.fix) {
        nf = std::max<int64_t>(nf, f.ntri);
        for (const PairPanel &l : P.lane) P.pairs += (int64_t)f.ntri * l.ntri;
    }
    P.work = std::max<size_t>(256, (size_t)nf * (size_t)nl * per);
}

bool pairs_touch(const bem_mesh &m, const PairPlan &P)
{
    std::vector<char> mark((size_t)m.nv, 0);
    for (const PairPanel &l : P.lane)
        for (int32_t i = 0; i < l.ntri; ++i)
            for (int a = 0; a < 3; ++a) mark[m.tri[3 * (size_t)P.ints[l.tri + i] + a]] = 1;
    for (const PairPanel &f : P.fix)
        for (int32_t i = 0; i < f.ntri; ++i)
            for (int a = 0; a < 3; ++a)
                if (mark[m.tri[3 * (size_t)P.ints[f.tri + i] + a]]) return true;
    return false;
}

namespace {

// Number of panels cut_side makes of `distinct` triangles with at most `most` a
// panel: neighbouring panels repeat the triangles on the line between them, about
// 2 sqrt(most) a panel.  repeat: by how much that makes them more.
double panel_count(int64_t distinct, int64_t most, double &repeat)
{
    repeat = 1.0;
    if (distinct <= most) return 1.0;
    repeat = 1.0 / std::max(0.5, 1.0 - 2.0 / std::sqrt((double)most));
    return std::ceil((double)distinct * repeat / (double)most);
}

// What one triangle pair costs by stars, what its local matrix and one star
// product of an entry's gather cost by pairs (picoseconds), and what a panel's two
// launches and its half-empty gather take at least (microseconds).
struct FormCost {
    double star, local, gather, panel;
};

FormCost form_cost(bool fp32, bool cplx, int q)
{
    if (q == 6) {
        if (fp32) return cplx ? FormCost{28.6, 53.0, 2.9, 29.0} : FormCost{12.4, 24.0, 1.44, 26.0};
        return cplx ? FormCost{57.0, 104.0, 5.5, 35.0} : FormCost{22.7, 42.0, 2.6, 21.0};
    }
    if (fp32) return cplx ? FormCost{16.3, 36.0, 2.9, 29.0} : FormCost{8.4, 19.0, 1.44, 26.0};
    return cplx ? FormCost{28.7, 62.0, 5.5, 35.0} : FormCost{13.1, 30.0, 2.6, 21.0};
}

}  // namespace

// By pairs a block costs its distinct triangle pairs' local matrices and its
// entries' gathers, by stars each fixed dof's star against the lanes of every
// chunk; chunks of more than 256 lanes repeat about a quarter of their triangles
// at the borders.  The costs above are those of two patches of 3,000 x 4,000
// vertices with all the workspace they want (us by stars / by pairs, 6-point rule:
// FP32 2,300 / 1,884, complex 5,316 / 3,983, FP64 4,212 / 3,269, complex 10,588 /
// 7,667; 4-point rule 1,564 / 1,600, 3,026 / 3,095, 2,439 / 2,645, 5,335 / 5,560:
// with fewer points a pair the matrices' way through memory outweighs what they
// save).  A small workspace cuts the block into panels (1,023 x 2,049, 6 points, by
// stars, by pairs in 16, 64 and 256 MiB: FP32 494, 999, 466, 391; complex 1,031,
// 3,421, 916, 761; FP64 810, 2,681, 771, 647; complex 1,916, 6,033, 1,972, 1,327).
// Scattered dofs share nothing and stay with the stars (two sets of 1,024: 377 us
// by stars, 554 by pairs), and so do blocks too small for two launches (two
// patches of n vertices, FP32 n = 400 72 / 81, 600 115 / 104; complex 200 75 / 71,
// 400 118 / 100; FP64 200 66 / 63, 400 99 / 90; complex 128 38 / 51, 200 121 / 82)
// and discontinuous dofs, whose stars are one triangle (1,023 x 2,049 FP32 95 /
// 113, FP64 108 / 140; 6,000 x 12,000 1,597 / 2,051 and 1,992 / 2,420).
// Served requests differ in where the entries go: the star kernels store them one
// by one over the host link in the caller's order (0.85 ns each), by pairs they
// are gathered on the device and copied (50 GB/s): 1,023 x 2,049 served, 16 MiB,
// FP32 2,316 / 1,384, complex 2,882 / 4,037, FP64 2,658 / 3,326, complex
// 3,015 / 7,163; 600 x 600 506 / 325, 666 / 580, 625 / 511, 761 / 1,189; discontinuous
// 600 x 600 FP32 144 / 162, FP64 200 / 215, 1,023 x 2,049 1,688 / 463, 1,830 / 688.
bool pairs_pay(const Request &r, const std::vector<int32_t> &fix, const std::vector<int32_t> &lane, const PairRoom &room)
{
    const bool fp32 = r.prec == BEM_FP32, cplx = is_complex_op(r.op);
    const double entries = (double)fix.size() * (double)lane.size();
    const double least = r.space == BEM_DP1 ? 524288 : fp32 ? (cplx ? 65536 : 262144) : (cplx ? 32768 : 65536);
    if (r.space == BEM_P0 || (r.space == BEM_DP1 && !room.served) || fix.size() < 8 || entries < least) return false;
    const bem_mesh &m = *r.mesh;
    const size_t per = pair_bytes(r.op, r.prec);
    const PanelCut cut = panel_cut(m, room.budget / per);
    int64_t fs, fd, ls, ld;
    count_side(m, r.space, fix.data(), (int64_t)fix.size(), fs, fd);
    count_side(m, r.space, lane.data(), (int64_t)lane.size(), ls, ld);
    double frep, lrep;
    const double lpan = panel_count(ld, cut.lanes, lrep);
    const double panels = lpan * panel_count(fd, cut.fixed(std::min(ld, cut.lanes)), frep);
    const FormCost c = form_cost(fp32, cplx, m.q);
    double star = 1e-6 * c.star * (double)fs * (ld > kBlockLanes ? 1.25 : 1.0) * (double)ld;
    double pair = 1e-6 * c.local * (double)fd * frep * (double)ld * lrep +
                  std::max(1e-6 * c.gather * (double)fs * (double)ls, c.panel * (panels - 1.0));
    if (room.served) {
        star += 0.85e-3 * entries;
        pair += 20e-6 * entries * (double)out_elem_bytes(r.op, r.prec);
    }
    return pair < 0.95 * star;
}

hipError_t launch_pairs(const bem_mesh &m, const PairPlan &P, const PairPanel &f, const PairPanel &l, const int32_t *ints,
                        void *work, void *out, int64_t sf, int64_t sl, double k, hipStream_t s, bool in_panel,
                        hipEvent_t between)
{
    const bool fp32 = P.prec == BEM_FP32, cplx = is_complex_op(P.op);
    void *Li = cplx ? static_cast<char *>(work) + (size_t)f.ntri * (size_t)l.ntri * pair_bytes(P.op, P.prec) / 2 : nullptr;
    hipError_t e = launch_pair_local(P.op, fp32, P.ltrial, m, ints + f.tri, f.ntri, ints + l.tri, l.ntri, work, Li, k, s);
    if (e == hipSuccess && between) e = hipEventRecord(between, s);
    if (e != hipSuccess) return e;
    return launch_pair_gather(fp32, cplx, work, Li, l.ntri, ints + f.ptr, ints + f.src, in_panel ? nullptr : ints + f.pos, f.ndof,
                              ints + l.ptr, ints + l.src, ints + l.pos, l.ndof, out, sf, sl, s);
}

namespace {

// Output panels in flight: one being computed, one on its way to the host, one
// being copied into the result.
constexpr int kPanels = 3;

// What a dense assembly works in: its streams, events, device memory (indices,
// local matrices, output panels) and pinned memory.  Kept between calls, since
// taking it anew is most of a small block's time (834 x 736 in FP64, 1.1 ms of
// which the kernels are 0.2; where the driver puts off returning the memory,
// 5 ms; 0.5 with a kept kit): at most kKits, kKitBytes of device and kKitPinned of pinned memory
// together; the last mesh's end gives them back.
struct DenseKit {
    int device = 0;
    char *dev = nullptr, *pin = nullptr;
    size_t dev_bytes = 0, pin_bytes = 0;
    hipStream_t sc = nullptr, sx = nullptr;
    hipEvent_t computed[kPanels] = {}, copied[kPanels] = {}, timed[3] = {};
    ~DenseKit()
    {
        for (hipEvent_t e : computed)
            if (e) (void)hipEventDestroy(e);
        for (hipEvent_t e : copied)
            if (e) (void)hipEventDestroy(e);
        for (hipEvent_t e : timed)
            if (e) (void)hipEventDestroy(e);
        if (sc) (void)hipStreamDestroy(sc);
        if (sx) (void)hipStreamDestroy(sx);
        if (dev) (void)hipFree(dev);
        if (pin) (void)hipHostFree(pin);
    }
};
constexpr size_t kKits = 4, kKitBytes = size_t(1536) << 20, kKitPinned = size_t(256) << 20;
std::mutex g_kit_mu;
// idle ones (never destroyed: at the process's end the runtime may be gone)
std::vector<std::unique_ptr<DenseKit>> &g_kits = *new std::vector<std::unique_ptr<DenseKit>>();

hipError_t take_kit(size_t dev_bytes, size_t pin_bytes, std::unique_ptr<DenseKit> &kit)
{
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    {
        std::lock_guard<std::mutex> g(g_kit_mu);
        size_t best = g_kits.size();   // the largest one
        for (size_t i = 0; i < g_kits.size(); ++i)
            if (g_kits[i]->device == device && (best == g_kits.size() || g_kits[i]->dev_bytes > g_kits[best]->dev_bytes)) best = i;
        if (best < g_kits.size()) {
            kit = std::move(g_kits[best]);
            g_kits.erase(g_kits.begin() + (std::ptrdiff_t)best);
        }
    }
    if (!kit) {
        kit.reset(new DenseKit());
        kit->device = device;
        e = hipStreamCreateWithFlags(&kit->sc, hipStreamNonBlocking);
        if (e == hipSuccess) e = hipStreamCreateWithFlags(&kit->sx, hipStreamNonBlocking);
        for (int i = 0; i < kPanels && e == hipSuccess; ++i) {
            e = hipEventCreateWithFlags(&kit->computed[i], hipEventDisableTiming);
            if (e == hipSuccess) e = hipEventCreateWithFlags(&kit->copied[i], hipEventDisableTiming);
        }
        for (int i = 0; i < 3 && e == hipSuccess; ++i) e = hipEventCreateWithFlags(&kit->timed[i], 0);
    }
    if (e == hipSuccess && kit->dev_bytes < dev_bytes) {
        if (kit->dev) (void)hipFree(kit->dev);
        kit->dev = nullptr;
        kit->dev_bytes = 0;
        e = hipMalloc((void **)&kit->dev, dev_bytes);
        if (e == hipSuccess) kit->dev_bytes = dev_bytes;
    }
    if (e == hipSuccess && kit->pin_bytes < pin_bytes) {
        if (kit->pin) (void)hipHostFree(kit->pin);
        kit->pin = nullptr;
        kit->pin_bytes = 0;
        e = hipHostMalloc((void **)&kit->pin, pin_bytes, hipHostMallocDefault);
        if (e == hipSuccess) kit->pin_bytes = pin_bytes;
    }
    return e;
}

// The kit's streams are idle.  One whose work failed is not kept.
void give_kit(std::unique_ptr<DenseKit> kit, bool keep)
{
    std::vector<std::unique_ptr<DenseKit>> gone;
    std::lock_guard<std::mutex> g(g_kit_mu);
    if (!keep || kit->dev_bytes > kKitBytes || kit->pin_bytes > kKitPinned) return;
    g_kits.push_back(std::move(kit));
    auto over = [&] {
        size_t d = 0, p = 0;
        for (const auto &x : g_kits) {
            d += x->dev_bytes;
            p += x->pin_bytes;
        }
        return g_kits.size() > kKits || d > kKitBytes || p > kKitPinned;
    };
    while (over()) {   // the one unused for longest
        gone.push_back(std::move(g_kits.front()));
        g_kits.erase(g_kits.begin());
    }
}

}  // namespace

void release_dense_kits()
{
    std::vector<std::unique_ptr<DenseKit>> gone;
    std::lock_guard<std::mutex> g(g_kit_mu);
    gone.swap(g_kits);
}

int eval_dense(bem_mesh *m, int op, int space, double k, const int32_t *rows, int64_t nrows, const int32_t *cols,
               int64_t ncols, int prec, int near, void *out, bem_dense_stats *st)
{
    if (!m) return fail(BEM_E_ARG, "null mesh");
    if (nrows < 0 || ncols < 0 || (nrows > 0 && !rows) || (ncols > 0 && !cols)) return fail(BEM_E_ARG, "bad indices");
    {
        Request probe;   // validates operator, space, k, precision and policy
        probe.mesh = m;
        probe.op = op;
        probe.space = space;
        probe.prec = prec;
        probe.k = k;
        probe.near = near;
        const int rc = expand_request(probe);
        if (rc != BEM_OK) return rc;
    }
    if (space != BEM_P1) return fail(BEM_E_ARG, "pair-based blocks are P1 only");
    if (op != BEM_LAPLACE_SLP && op != BEM_LAPLACE_DLP && op != BEM_HELMHOLTZ_SLP && op != BEM_HELMHOLTZ_DLP)
        return fail(BEM_E_ARG, "pair-based blocks: single and double layer only");
    if (near == BEM_NEAR_SINGULAR) return fail(BEM_E_ARG, "pair-based blocks: BEM_NEAR_ERROR or BEM_NEAR_SKIP");
    for (int64_t i = 0; i < nrows; ++i)
        if (rows[i] < 0 || rows[i] >= m->nv) return fail(BEM_E_ARG, "row index out of range");
    for (int64_t i = 0; i < ncols; ++i)
        if (cols[i] < 0 || cols[i] >= m->nv) return fail(BEM_E_ARG, "column index out of range");
    if (st) *st = bem_dense_stats{};
    if (nrows == 0 || ncols == 0) return BEM_OK;
    if (ncols > INT32_MAX / 4) return fail(BEM_E_ARG, "too many columns");
    const double t0 = now_seconds();
    const size_t elem = out_elem_bytes(op, prec);

    // row panels whose local matrices take at most BEM_DENSE_BUDGET_MB (default 1024) MiB
    const char *env = std::getenv("BEM_DENSE_BUDGET_MB");
    const size_t budget = (size_t)std::max(16, env ? std::atoi(env) : 1024) << 20;
    PairPlan P;
    plan_pairs(*m, space, op, prec, true, rows, nrows, cols, ncols, budget, P, true);
    // nothing is launched for a failing request
    if (near == BEM_NEAR_ERROR && pairs_touch(*m, P))
        return fail(BEM_E_NEARFIELD, "a contributing triangle pair shares a vertex");
    int64_t stars, ntrial, longest = 0;
    count_side(*m, space, cols, ncols, stars, ntrial);
    for (int64_t i = 0; i < nrows; ++i) longest = std::max(longest, m->star_ptr[rows[i] + 1] - m->star_ptr[rows[i]]);
    if ((size_t)longest * (size_t)ntrial * pair_bytes(op, prec) > budget)
        return fail(BEM_E_OOM, "one row's local matrices exceed the dense budget (BEM_DENSE_BUDGET_MB)");
    const std::vector<PairPanel> &panels = P.fix;
    int64_t max_rows = 0;
    for (const PairPanel &f : panels) max_rows = std::max<int64_t>(max_rows, f.ndof);
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t row_bytes = (size_t)ncols * elem, panel_out = al((size_t)max_rows * row_bytes);
    const size_t ints = al(4 * P.ints.size());
    size_t bufs = std::min<size_t>(kPanels, panels.size());
    std::unique_ptr<DenseKit> kit;
    hipError_t e;
    for (;; --bufs) {
        e = take_kit(ints + al(P.work) + bufs * panel_out, ints + bufs * panel_out, kit);
        if (e != hipErrorOutOfMemory || bufs == 1) break;
        (void)hipGetLastError();
        kit.reset();             // with less, and without what other calls left
        release_kept();
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(e == hipErrorOutOfMemory ? BEM_E_OOM : BEM_E_DEVICE, std::string("dense set-up: ") + hipGetErrorString(e));
    }
    const hipStream_t sc = kit->sc, sx = kit->sx;
    char *d_L = kit->dev + ints, *d_out = d_L + al(P.work), *h_out = kit->pin + ints;
    const int32_t *D = reinterpret_cast<const int32_t *>(kit->dev);
    std::memcpy(kit->pin, P.ints.data(), 4 * P.ints.size());
    e = hipMemcpyAsync(kit->dev, kit->pin, 4 * P.ints.size(), hipMemcpyHostToDevice, sc);

    // a panel's rows, where the caller has them, about a MiB at a time
    const int64_t per = std::max<int64_t>(1, (int64_t)((size_t(1) << 20) / row_bytes));
    std::vector<int64_t> first(1, 0);   // per panel its first part
    for (const PairPanel &f : panels) first.push_back(first.back() + (f.ndof + per - 1) / per);
    auto part = [&](int64_t i) {
        const size_t p = (size_t)(std::upper_bound(first.begin(), first.end(), i) - first.begin()) - 1;
        const PairPanel &f = panels[p];
        const char *src = h_out + p % bufs * panel_out;
        const int64_t r0 = (i - first[p]) * per, r1 = std::min<int64_t>(f.ndof, r0 + per);
        for (int64_t r = r0; r < r1; ++r)
            std::memcpy(static_cast<char *>(out) + (size_t)P.ints[f.pos + r] * row_bytes, src + (size_t)r * row_bytes, row_bytes);
    };
    {
        CopyCrew<decltype(part)> crew(copy_helpers((size_t)nrows * row_bytes, 7), part);
        auto enqueue = [&](size_t p) {
            const PairPanel &f = panels[p];
            const size_t b = p % bufs;
            char *dout = d_out + b * panel_out;
            hipError_t x = hipSuccess;
            if (p == 0) x = hipEventRecord(kit->timed[0], sc);
            // the panel that had this buffer has been copied out: its transfer has ended
            for (size_t l = 0; l < P.lane.size() && x == hipSuccess; ++l)
                x = launch_pairs(*m, P, f, P.lane[l], D, d_L, dout, ncols, 1, k, sc, true,
                                 p == 0 && l == 0 ? kit->timed[1] : nullptr);
            if (x == hipSuccess && p == 0) x = hipEventRecord(kit->timed[2], sc);
            if (x == hipSuccess) x = hipEventRecord(kit->computed[b], sc);
            if (x == hipSuccess) x = hipStreamWaitEvent(sx, kit->computed[b], 0);
            if (x == hipSuccess)
                x = hipMemcpyAsync(h_out + b * panel_out, dout, (size_t)f.ndof * row_bytes, hipMemcpyDeviceToHost, sx);
            if (x == hipSuccess) x = hipEventRecord(kit->copied[b], sx);
            return x;
        };
        size_t ahead = 0;
        for (size_t p = 0; p < panels.size() && e == hipSuccess; ++p) {
            while (ahead < panels.size() && ahead < p + bufs && e == hipSuccess) {
                if (ahead >= bufs) crew.help(first[ahead - bufs + 1]);
                e = enqueue(ahead++);
            }
            if (e == hipSuccess) e = hipEventSynchronize(kit->copied[p % bufs]);
            if (e == hipSuccess) crew.release(first[p + 1]);
        }
        if (e == hipSuccess) crew.help(first.back());
    }
    if (st && e == hipSuccess) {   // the first panel's kernel times
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, kit->timed[0], kit->timed[1]) == hipSuccess) st->first_local_seconds = 1e-3 * ms;
        if (hipEventElapsedTime(&ms, kit->timed[1], kit->timed[2]) == hipSuccess) st->first_gather_seconds = 1e-3 * ms;
        st->first_pairs = (int64_t)panels[0].ntri * P.lane[0].ntri;
    }
    int rc = BEM_OK;
    if (e != hipSuccess) {
        rc = fail(BEM_E_DEVICE, std::string("dense block: ") + hipGetErrorString(e));
        (void)hipStreamSynchronize(sc);
        (void)hipStreamSynchronize(sx);
    }
    give_kit(std::move(kit), rc == BEM_OK);
    if (st && rc == BEM_OK) {
        st->pairs = P.pairs;
        st->panels = (int64_t)panels.size();
        st->seconds = now_seconds() - t0;
    }
    return rc;
}

}  // namespace bem
