// P1 and DP1 blocks by triangle pairs (the dense weak-form assembly of
// Section 3): every regular triangle pair of star(rows) x star(cols) is
// integrated once into its 3 x 3 local matrix on the device, then each entry
// adds its pairs' local values in a fixed order (entries.hip: k_local_*,
// k_gather_pairs).  Device-tensor requests large enough take it
// (pairs_pay); bem_eval_dense is the host form: rows go in panels whose local
// matrices fit a device budget; the panels run on a compute stream while a
// copy stream moves the previous panel's entries to pinned host memory and the
// calling thread copies the one before into `out`, so assembly and transfer
// overlap (Section 3's chunked assembly with overlapped transfers).
#include <algorithm>
#include <cstdlib>

#include "bem_internal.hpp"

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
// star at least).
void cut_side(const bem_mesh &m, int space, const int32_t *dofs, int64_t n, int64_t most_tri, std::vector<int32_t> &ints,
              std::vector<PairPanel> &out)
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
            if (i > first && (int64_t)tri.size() + fresh > most_tri) break;
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
void count_side(const bem_mesh &m, int space, const std::vector<int32_t> &dofs, int64_t &stars, int64_t &distinct)
{
    PairScratch &sc = g_pair;
    sc.open(m.nt);
    stars = distinct = 0;
    for (int32_t d : dofs) {
        int64_t b, e;
        star_range(m, space, d, b, e);
        stars += e - b;
        for (int64_t s = b; s < e; ++s) {
            const int32_t t = m.star[s] >> 2;
            distinct += sc.stamp[t] != sc.gen;
            sc.stamp[t] = sc.gen;
        }
    }
}

size_t pair_bytes(int op, int prec) { return 9 * (prec == BEM_FP32 ? 4 : 8) * (size_t)(is_complex_op(op) ? 2 : 1); }

}  // namespace

void plan_pairs(const bem_mesh &m, int space, int op, int prec, bool ltrial, const int32_t *fix, int64_t nfix,
                const int32_t *lane, int64_t nlane, size_t budget, PairPlan &P)
{
    P.ints.clear();
    P.fix.clear();
    P.lane.clear();
    P.op = op;
    P.prec = prec;
    P.ltrial = ltrial;
    const size_t per = pair_bytes(op, prec);
    // lane panels leave room for at least 64 fixed-side triangles (or the largest star)
    const int64_t rows = std::max<int64_t>(64, m.max_star);
    cut_side(m, space, lane, nlane, std::max<int64_t>(256, (int64_t)(budget / per) / rows), P.ints, P.lane);
    int64_t nl = 1;
    for (const PairPanel &l : P.lane) nl = std::max<int64_t>(nl, l.ntri);
    // 262,144 rows: the launch grid's second dimension at four or more rows a workgroup
    cut_side(m, space, fix, nfix, std::min<int64_t>(std::max<int64_t>(1, (int64_t)(budget / per) / nl), 65535 * 4), P.ints,
             P.fix);
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

// By pairs a block costs its distinct triangle pairs' local matrices and its
// entries' gathers, by stars each fixed dof's star against the lanes of every
// chunk.  Per point pair a local matrix takes 11 instructions to the star
// form's 9 (6-point rule, single layer; with the basis products of the pair 1.3
// times a star pair's), a gather a tenth of a star pair for each of an entry's
// star products.  Chunks of more than 256 lanes repeat about a quarter of their
// triangles at the borders.  Scattered dofs share nothing and stay with the
// stars (two sets of 1,024: 377 us by stars, 554 by pairs).  Small blocks stay
// with them too, for their single launch; the line is where the two meet for
// two patches of n dofs (us by stars / by pairs): FP32 n = 362 39 / 56, 512
// 63 / 65, 1,024 191 / 128; FP32 complex 256 65 / 62, 1,024 451 / 330; FP64 256
// 55 / 49, 1,024 344 / 252; FP64 complex 128 38 / 51, 181 80 / 58, 1,024
// 970 / 641.
bool pairs_pay(const Request &r, const std::vector<int32_t> &fix, const std::vector<int32_t> &lane)
{
    const bool fp32 = r.prec == BEM_FP32, cplx = is_complex_op(r.op);
    const int64_t least = fp32 ? (cplx ? 65536 : 262144) : (cplx ? 32768 : 65536);
    if (r.space == BEM_P0 || fix.size() < 8 || (int64_t)fix.size() * (int64_t)lane.size() < least) return false;
    const bem_mesh &m = *r.mesh;
    int64_t fs, fd, ls, ld;
    count_side(m, r.space, fix, fs, fd);
    count_side(m, r.space, lane, ls, ld);
    const double star = (double)fs * (ld > kBlockLanes ? 1.25 : 1.0) * (double)ld;
    const double pair = 1.3 * (double)fd * (double)ld + 0.1 * (double)fs * (double)ls;
    return pair < 0.8 * star;
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

struct DevBuf {
    void *p = nullptr;
    ~DevBuf()
    {
        if (p) (void)hipFree(p);
    }
};

}  // namespace

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
    plan_pairs(*m, space, op, prec, true, rows, nrows, cols, ncols, budget, P);
    // nothing is launched for a failing request
    if (near == BEM_NEAR_ERROR && pairs_touch(*m, P))
        return fail(BEM_E_NEARFIELD, "a contributing triangle pair shares a vertex");
    const std::vector<PairPanel> &panels = P.fix;
    int64_t max_rows = 0;
    for (const PairPanel &f : panels) max_rows = std::max<int64_t>(max_rows, f.ndof);
    const size_t panel_out = (size_t)max_rows * (size_t)ncols * elem;
    DevBuf d_idx, d_L, d_out;
    char *h_stage = nullptr;
    hipStream_t sc = nullptr, sx = nullptr;
    hipEvent_t ev[8] = {};
    int rc = BEM_OK;
    auto cleanup = [&]() {
        if (sc) (void)hipStreamSynchronize(sc);
        if (sx) (void)hipStreamSynchronize(sx);
        for (hipEvent_t e : ev)
            if (e) (void)hipEventDestroy(e);
        if (sc) (void)hipStreamDestroy(sc);
        if (sx) (void)hipStreamDestroy(sx);
        if (h_stage) (void)hipHostFree(h_stage);
    };
    hipError_t e = hipMalloc(&d_idx.p, 4 * P.ints.size());
    if (e == hipSuccess) e = hipMalloc(&d_L.p, P.work);
    if (e == hipSuccess) e = hipMalloc(&d_out.p, 2 * panel_out);
    if (e == hipSuccess) e = hipHostMalloc((void **)&h_stage, 2 * panel_out, hipHostMallocDefault);
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&sc, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&sx, hipStreamNonBlocking);
    for (int i = 0; i < 8 && e == hipSuccess; ++i) e = hipEventCreateWithFlags(&ev[i], i < 4 ? hipEventDisableTiming : 0);
    if (e == hipSuccess) e = hipMemcpy(d_idx.p, P.ints.data(), 4 * P.ints.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        cleanup();
        return fail(e == hipErrorOutOfMemory ? BEM_E_OOM : BEM_E_DEVICE, std::string("dense set-up: ") + hipGetErrorString(e));
    }
    const int32_t *D = static_cast<const int32_t *>(d_idx.p);
    hipEvent_t *computed = ev, *copied = ev + 2;   // per output buffer
    hipEvent_t t_start = ev[4], t_local = ev[5], t_end = ev[6];
    double local_s = 0.0;
    auto finish = [&](size_t p) {
        const PairPanel &f = panels[p];
        const int b = (int)(p % 2);
        hipError_t x = hipEventSynchronize(copied[b]);
        if (x != hipSuccess) return x;
        for (int32_t r = 0; r < f.ndof; ++r)   // the panel's rows, where the caller has them
            std::memcpy(static_cast<char *>(out) + (size_t)P.ints[f.pos + r] * ncols * elem,
                        h_stage + b * panel_out + (size_t)r * ncols * elem, (size_t)ncols * elem);
        return hipSuccess;
    };
    for (size_t p = 0; p < panels.size() && e == hipSuccess; ++p) {
        const PairPanel &f = panels[p];
        const int b = (int)(p % 2);
        char *dout = static_cast<char *>(d_out.p) + b * panel_out;
        if (p >= 2) e = hipStreamWaitEvent(sc, copied[b], 0);
        const bool timed = p == 0;
        if (e == hipSuccess && timed) e = hipEventRecord(t_start, sc);
        for (size_t l = 0; l < P.lane.size() && e == hipSuccess; ++l)
            e = launch_pairs(*m, P, f, P.lane[l], D, d_L.p, dout, ncols, 1, k, sc, true,
                             timed && l == 0 ? t_local : nullptr);
        if (e == hipSuccess && timed) e = hipEventRecord(t_end, sc);
        if (e == hipSuccess) e = hipEventRecord(computed[b], sc);
        if (e == hipSuccess && p >= 1) e = finish(p - 1);
        if (e == hipSuccess) e = hipStreamWaitEvent(sx, computed[b], 0);
        if (e == hipSuccess)
            e = hipMemcpyAsync(h_stage + b * panel_out, dout, (size_t)f.ndof * ncols * elem, hipMemcpyDeviceToHost, sx);
        if (e == hipSuccess) e = hipEventRecord(copied[b], sx);
        if (e == hipSuccess && timed) {
            float ms0 = 0.f;
            // the first panel's kernel times (one synchronisation, at the end of the first panel)
            if (hipEventSynchronize(t_end) == hipSuccess && hipEventElapsedTime(&ms0, t_start, t_local) == hipSuccess)
                local_s = 1e-3 * ms0;
            if (st) {
                float ms1 = 0.f;
                if (hipEventElapsedTime(&ms1, t_local, t_end) == hipSuccess) st->first_gather_seconds = 1e-3 * ms1;
                st->first_local_seconds = local_s;
                st->first_pairs = (int64_t)f.ntri * P.lane[0].ntri;
            }
        }
    }
    if (e == hipSuccess) e = finish(panels.size() - 1);
    if (e != hipSuccess) rc = fail(BEM_E_DEVICE, std::string("dense block: ") + hipGetErrorString(e));
    cleanup();
    if (st && rc == BEM_OK) {
        st->pairs = P.pairs;
        st->panels = (int64_t)panels.size();
        st->seconds = now_seconds() - t0;
    }
    return rc;
}

}  // namespace bem
