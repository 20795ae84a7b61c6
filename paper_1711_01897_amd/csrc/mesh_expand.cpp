// Mesh residency and request expansion (host side).
//
// A request A[rows, cols] becomes work for the entry kernels:
//  * P0 (dof = triangle): entry (i, j) is the single triangle pair (T_i, T_j).
//    The longer of the two index lists runs across the lanes of a workgroup
//    (in chunks of 256), the other one is the workgroup's fixed side.
//  * P1 (dof = vertex, hat functions, Section 2): entry (I, J) sums over the
//    triangles m around I and n around J.  With the column side on the lanes,
//    the requested columns are cut into runs whose stars together hold at
//    most 256 triangles; each run's triangles form one chunk of lanes, every
//    lane triangle serving each of its requested vertices in the run, and the
//    fixed side of a workgroup is the star of one row vertex.  A segment list
//    maps every requested column to its (lane triangle, local vertex) partial
//    sums in ascending triangle order, which fixes the order of the final
//    per-entry sum.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <string>

#include "bem_internal.hpp"

namespace bem {

namespace {
thread_local std::string g_last_error;
}

void set_error(const std::string &msg) { g_last_error = msg; }

int fail(int code, const std::string &msg)
{
    g_last_error = msg;
    return code;
}

const char *last_error() { return g_last_error.c_str(); }

double now_seconds()
{
    using clk = std::chrono::steady_clock;
    return std::chrono::duration<double>(clk::now().time_since_epoch()).count();
}

bool is_complex_op(int op)
{
    return op == BEM_HELMHOLTZ_SLP || op == BEM_HELMHOLTZ_DLP || op == BEM_HELMHOLTZ_ADLP || op == BEM_HELMHOLTZ_HYPS;
}

bool is_adjoint_op(int op) { return op == BEM_LAPLACE_ADLP || op == BEM_HELMHOLTZ_ADLP; }

int64_t space_ndof(const bem_mesh &m, int space)
{
    return space == BEM_P0 ? m.nt : (space == BEM_P1 ? m.nv : 3 * m.nt);
}

int kernel_op(int op)
{
    if (op == BEM_LAPLACE_ADLP) return BEM_LAPLACE_DLP;
    if (op == BEM_HELMHOLTZ_ADLP) return BEM_HELMHOLTZ_DLP;
    return op;
}

size_t out_elem_bytes(int op, int prec)
{
    const size_t real = prec == BEM_FP32 ? 4 : 8;
    return is_complex_op(op) ? 2 * real : real;
}

namespace {

// Per-thread scratch mapping triangles to lane slots.
struct StarScratch {
    std::vector<int32_t> slot_of;
    std::vector<uint32_t> stamp;
    uint32_t gen = 0;
    void prepare(int64_t nt)
    {
        if ((int64_t)stamp.size() < nt) {
            stamp.assign(nt, 0);
            slot_of.assign(nt, -1);
            gen = 0;
        }
        next_gen();
    }
    void next_gen()
    {
        if (++gen == 0) {
            std::fill(stamp.begin(), stamp.end(), 0);
            gen = 1;
        }
    }
};
thread_local StarScratch g_scratch;

size_t align16(size_t x) { return (x + 15) & ~(size_t)15; }

void expand_fixed(const bem_mesh &m, int space, const int32_t *dofs, int64_t n, Request &r)
{
    r.fix.clear();
    r.nstar = 0;
    if (space == BEM_P0) {
        r.fix.assign(dofs, dofs + n);
    } else if (space == BEM_P1) {
        // the fixed dofs' stars stay in the mesh's star table: ranges only
        r.fix.resize(2 * n);
        for (int64_t f = 0; f < n; ++f) {
            const int32_t v = dofs[f];
            r.fix[2 * f] = (int32_t)m.star_ptr[v];
            r.fix[2 * f + 1] = (int32_t)m.star_ptr[v + 1];
            r.nstar += m.star_ptr[v + 1] - m.star_ptr[v];
        }
    } else {
        // DP1: a dof is the one-triangle star (t, a), one entry of the star table
        r.fix.resize(2 * n);
        for (int64_t f = 0; f < n; ++f) {
            r.fix[2 * f] = m.dp1_star[dofs[f]];
            r.fix[2 * f + 1] = r.fix[2 * f] + 1;
        }
        r.nstar = n;
    }
    r.nfix = n;
}

void finalize_sizes(Request &r)
{
    const bem_mesh &m = *r.mesh;
    const int64_t q2 = (int64_t)m.q * m.q;
    r.elem_bytes = out_elem_bytes(r.op, r.prec);
    const int64_t fixed_tris = r.space == BEM_P0 ? r.nfix : r.nstar;
    r.evals = fixed_tris * r.ndistinct * q2;
    r.nblocks = (r.nfix + r.tile - 1) / r.tile * r.nchunk;
    const size_t own = r.ext ? 0 : r.own.ints() + (r.tile > 1 ? r.fix.size() : 0);
    r.in_bytes = align16(4 * own);
    r.out_bytes = align16((size_t)r.entries() * r.elem_bytes);
    r.batch_bytes = request_bytes(r);
}

}  // namespace

namespace {

// 30-bit Morton code of a point in the mesh's bounding box (10 bits per axis).
uint32_t morton3(double x, double y, double z, const double *lo, const double *inv)
{
    auto spread = [](uint32_t v) {
        v &= 1023u;
        v = (v | (v << 16)) & 0x030000FFu;
        v = (v | (v << 8)) & 0x0300F00Fu;
        v = (v | (v << 4)) & 0x030C30C3u;
        v = (v | (v << 2)) & 0x09249249u;
        return v;
    };
    auto q = [](double t) { return (uint32_t)std::min(1023.0, std::max(0.0, t * 1023.0)); };
    return spread(q((x - lo[0]) * inv[0])) | (spread(q((y - lo[1]) * inv[1])) << 1) |
           (spread(q((z - lo[2]) * inv[2])) << 2);
}

}  // namespace

void morton_order(const bem_mesh &m, int space, const int32_t *dofs, int64_t n, std::vector<int32_t> &order)
{
    std::vector<std::pair<uint32_t, int32_t>> key((size_t)n);
    for (int64_t i = 0; i < n; ++i) {
        // P1: the vertex; DP1: the first vertex of the dof's triangle
        const int32_t v = space == BEM_P1 ? dofs[i] : m.tri[3 * (size_t)(dofs[i] / 3)];
        const double *x = &m.xyz[3 * (size_t)v];
        key[i] = {morton3(x[0], x[1], x[2], m.box_lo, m.box_inv), (int32_t)i};
    }
    std::sort(key.begin(), key.end());
    order.resize((size_t)n);
    for (int64_t i = 0; i < n; ++i) order[i] = key[i].second;
}

void build_lane_set(const bem_mesh &m, int space, const int32_t *dofs, int64_t n, LaneSet &ls, bool reorder)
{
    ls.pos.clear();
    if (reorder && space != BEM_P0 && n > kBlockLanes) {
        morton_order(m, space, dofs, n, ls.pos);
        std::vector<int32_t> sorted((size_t)n);
        for (int64_t i = 0; i < n; ++i) sorted[i] = dofs[ls.pos[i]];
        std::vector<int32_t> keep;
        keep.swap(ls.pos);
        build_lane_set(m, space, sorted.data(), n, ls, false);
        ls.pos.swap(keep);
        return;
    }
    ls.ndof = n;
    ls.lane.clear();
    ls.chunk.clear();
    ls.seg_ptr.clear();
    ls.seg.clear();
    if (space == BEM_P0) {
        ls.lane.assign(dofs, dofs + n);
        ls.ndistinct = n;
        for (int64_t c0 = 0; c0 < n; c0 += kBlockLanes) {
            const int32_t len = (int32_t)std::min<int64_t>(kBlockLanes, n - c0);
            ls.chunk.insert(ls.chunk.end(), {(int32_t)c0, len, (int32_t)c0, len});
        }
        return;
    }
    // P1: walk the dofs in order; a dof joins the open chunk while the
    // union of the chunk's stars stays within kBlockLanes triangles
    StarScratch &sc = g_scratch;
    sc.prepare(m.nt);
    ls.seg_ptr.resize(n + 1);
    ls.seg_ptr[0] = 0;
    int32_t lane0 = 0, count = 0;
    int64_t dof0 = 0;
    auto close = [&](int64_t end) {
        ls.chunk.insert(ls.chunk.end(), {lane0, count, (int32_t)dof0, (int32_t)(end - dof0)});
        lane0 += count;
        count = 0;
        dof0 = end;
        sc.next_gen();
    };
    // the star-table range of a dof: its vertex's star (P1) or the one entry
    // of its triangle and local vertex (DP1)
    auto range = [&](int32_t d, int64_t &b, int64_t &e) {
        if (space == BEM_P1) {
            b = m.star_ptr[d];
            e = m.star_ptr[d + 1];
        } else {
            b = m.dp1_star[d];
            e = b + 1;
        }
    };
    for (int64_t c = 0; c < n; ++c) {
        int64_t sb, se;
        range(dofs[c], sb, se);
        int32_t fresh = 0;
        for (int64_t s = sb; s < se; ++s) fresh += sc.stamp[m.star[s] >> 2] != sc.gen;
        if (count + fresh > kBlockLanes && c > dof0) close(c);
        for (int64_t s = sb; s < se; ++s) {
            const int32_t t = m.star[s] >> 2;
            if (sc.stamp[t] != sc.gen) {
                sc.stamp[t] = sc.gen;
                sc.slot_of[t] = count++;
                ls.lane.push_back(t);
            }
            ls.seg.push_back((sc.slot_of[t] << 2) | (m.star[s] & 3));
        }
        ls.seg_ptr[c + 1] = (int32_t)ls.seg.size();
    }
    if (n > dof0) close(n);
    // distinct triangles over all chunks
    ls.ndistinct = 0;
    for (int32_t t : ls.lane)
        if (sc.stamp[t] != sc.gen) {
            sc.stamp[t] = sc.gen;
            ++ls.ndistinct;
        }
    sc.next_gen();
}

namespace {

// P1 requests of few fixed dofs take the row form, whose lane side is the dof
// list itself: the star form's expansion of the lanes takes the host 62 ns for
// each of 4,096 dofs and 20 for each of 1,024, the row form's threads evaluate
// 2.4 times its pairs.  The line is where the two meet for 1,024 lane dofs, back
// to back on one stream (us by stars / by rows, 6-point rule): FP32 real 64 fixed
// dofs 42 / 41 (1: 39 / 19), complex 16 41 / 32, 32 43 / 48; FP64 real 16 41 / 28,
// 32 42 / 44; FP64 complex 8 44 / 36, 16 43 / 57.  Of 4,096 lane dofs all these
// are faster by rows (1: 259-271 / 21-24; the largest 283 / 124, 278 / 83,
// 275 / 71, 278 / 99), of 32 too (17-26 / 14-20).  The leaves of an H-matrix,
// which several threads expand while the device works on others, keep the star
// form (level-5 icosphere, leaf size 100: 58.5 ms by stars, 63 by rows); so do
// lists so long that the row form's block records, one for every 8 to 32 lane dofs
// where stars take one for about 100, exceed a workspace that the stars' fit.
bool row_pays(const Request &r, int64_t nfix)
{
    if (r.space == BEM_P0 || r.plain) return false;
    if (is_complex_op(r.op)) return nfix <= (r.prec == BEM_FP32 ? 16 : 8);
    return nfix <= (r.prec == BEM_FP32 ? 64 : 16);
}

// Lane side of the row form: the dofs (P1: vertices; DP1: star entries), in
// chunks of as many as a workgroup takes (32 vertices of eight threads, 256
// discontinuous dofs).  Where that gives fewer than 1,024 workgroups, a
// workgroup takes a half or a quarter of the vertices and its waves share the
// fixed star between them (FP64 Helmholtz, 32 dofs: 33 us a call with whole
// stars, 20 with quarters; from 1,024 workgroups on the two are alike).
void build_row_set(const bem_mesh &m, int space, int64_t nfix, const int32_t *dofs, int64_t n, LaneSet &ls,
                   int32_t &split)
{
    ls.pos.clear();
    ls.seg_ptr.clear();
    ls.seg.clear();
    ls.chunk.clear();
    ls.ndof = n;
    ls.lane.assign(dofs, dofs + n);
    if (space == BEM_DP1)
        for (int32_t &d : ls.lane) d = m.dp1_star[d];
    // a triangle counts for each of its requested vertices, as it is evaluated
    ls.ndistinct = n;
    if (space == BEM_P1) {
        ls.ndistinct = 0;
        for (int64_t d = 0; d < n; ++d) ls.ndistinct += m.star_ptr[dofs[d] + 1] - m.star_ptr[dofs[d]];
    }
    int64_t per = space == BEM_DP1 ? kBlockLanes : kBlockLanes / 8;
    split = 0;
    while (space == BEM_P1 && split < 2 && nfix * ((n + per - 1) / per) < 1024) {
        ++split;
        per /= 2;
    }
    for (int64_t c = 0; c < n; c += per) {
        const int32_t len = (int32_t)std::min<int64_t>(per, n - c);
        ls.chunk.insert(ls.chunk.end(), {(int32_t)c, len, (int32_t)c, len});
    }
}

// Largest distance of two points of triangles T and S (at two of their
// vertices).  The device writes x - y = rho c over a singular pair with the
// radius rho in [0, 1] and takes omega = k |c|; c is itself a difference x - y of
// points of the two triangles, at the corners of its domain of their vertices:
//   identical:     c runs along the three edge vectors;
//   common edge:   c = dh E + s1 a - s2 b on four faces;
//   common vertex: c = a(u) - z b(v) or z a(u) - b(v), u, v, z in [0, 1].
double near_span(const bem_mesh &m, int32_t T, int32_t S)
{
    double best = 0.0;
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            const double *x = &m.xyz[3 * (size_t)m.tri[3 * (size_t)T + i]], *y = &m.xyz[3 * (size_t)m.tri[3 * (size_t)S + j]];
            const double d0 = x[0] - y[0], d1 = x[1] - y[1], d2 = x[2] - y[2];
            best = std::max(best, std::sqrt(d0 * d0 + d1 * d1 + d2 * d2));
        }
    return best;
}

// The radial series (48 terms at most) of the Helmholtz singular pairs holds ~1e-14
// relative accuracy at omega = 6 and ~5e-10 at 12, then fails quickly (its
// largest terms grow like omega^n / n!): requests whose items reach beyond
// kOmegaMax are refused.
constexpr double kOmegaMax = 12.0;

int check_near_omega(const Request &r)
{
    // two triangles that share a vertex reach two edges at most
    if (!is_complex_op(r.op) || r.k * 2.0 * r.mesh->max_edge <= kOmegaMax) return BEM_OK;
    double span = 0.0;
    for (const NearPair &q : r.near_pairs) span = std::max(span, near_span(*r.mesh, q.a, q.b));
    if (r.k * span > kOmegaMax)
        return fail(BEM_E_ARG, "BEM_NEAR_SINGULAR Helmholtz pair with k |x - y| up to " + std::to_string(r.k * span) +
                                   " > 12: the singular scheme's radial series is accurate only below that (the mesh "
                                   "needs more than about one element per wavelength)");
    return BEM_OK;
}

// Per-thread marks of triangles and of column dofs (vertices or triangles).
struct NearScratch {
    std::vector<uint32_t> tri, col, slot;
    std::vector<int32_t> slot_of, head, next;
    uint32_t tgen = 0, cgen = 0, sgen = 0;
    static uint32_t fresh(std::vector<uint32_t> &v, uint32_t &gen, size_t n)
    {
        if (v.size() < n) {
            v.assign(n, 0);
            gen = 0;
        }
        if (++gen == 0) {
            std::fill(v.begin(), v.end(), 0);
            gen = 1;
        }
        return gen;
    }
};
thread_local NearScratch g_near;

bool same_pair_vanishes(const Request &r)
{
    // (x - y).n_y = 0 on a flat triangle
    return kernel_op(r.op) == BEM_LAPLACE_DLP || kernel_op(r.op) == BEM_HELMHOLTZ_DLP;
}

// The triangles that share a vertex with a, ascending, appended to out.
void neighbours(const bem_mesh &m, int32_t a, std::vector<int32_t> &out)
{
    NearScratch &sc = g_near;
    const uint32_t g = NearScratch::fresh(sc.tri, sc.tgen, (size_t)m.nt);
    out.clear();
    for (int k = 0; k < 3; ++k) {
        const int32_t v = m.tri[3 * (size_t)a + k];
        for (int64_t s = m.star_ptr[v]; s < m.star_ptr[v + 1]; ++s) {
            const int32_t b = m.star[s] >> 2;
            if (sc.tri[b] == g) continue;
            sc.tri[b] = g;
            out.push_back(b);
        }
    }
    std::sort(out.begin(), out.end());
}

// P0: one pair per entry whose two triangles share a vertex.
void build_near_p0(Request &r)
{
    const bem_mesh &m = *r.mesh;
    NearScratch &sc = g_near;
    const uint32_t cg = NearScratch::fresh(sc.col, sc.cgen, (size_t)std::max(m.nt, m.nv));
    if (sc.head.size() < sc.col.size()) sc.head.resize(sc.col.size());
    sc.next.resize((size_t)r.ncols);
    for (int64_t c = r.ncols - 1; c >= 0; --c) {   // positions of a column in ascending order
        const int32_t t = r.cols[c];
        sc.next[c] = sc.col[t] == cg ? sc.head[t] : -1;
        sc.col[t] = cg;
        sc.head[t] = (int32_t)c;
    }
    const bool skip_same = same_pair_vanishes(r);
    std::vector<int32_t> nb;
    for (int64_t i = 0; i < r.nrows; ++i) {
        const int32_t a = r.rows[i];
        neighbours(m, a, nb);
        for (int32_t b : nb) {
            if (sc.col[b] != cg || (skip_same && a == b)) continue;
            for (int32_t c = sc.head[b]; c >= 0; c = sc.next[c])
                r.near_pairs.push_back({a, b, 0, 0, i * r.ncols + c});
        }
    }
}

// P1 and DP1: the pairs (a, b) with a in the star of a requested row dof and
// b, adjacent to it, in the star of a requested column dof, grouped by a in
// the order the rows' stars name them, each once; the rows' stars as (group,
// local vertex).
void build_near_p1(Request &r)
{
    const bem_mesh &m = *r.mesh;
    const bool dp1 = r.space == BEM_DP1;
    NearScratch &sc = g_near;
    const uint32_t cg = NearScratch::fresh(sc.col, sc.cgen, (size_t)std::max(m.nt, m.nv));
    for (int32_t d : r.cols) sc.col[dp1 ? d / 3 : d] = cg;   // P1: vertices, DP1: triangles
    const uint32_t sg = NearScratch::fresh(sc.slot, sc.sgen, (size_t)m.nt);
    if (sc.slot_of.size() < (size_t)m.nt) sc.slot_of.resize((size_t)m.nt);
    const bool skip_same = same_pair_vanishes(r);
    std::vector<int32_t> nb, gptr{0}, rptr{0}, rs;
    rptr.reserve((size_t)r.nrows + 1);
    for (int64_t i = 0; i < r.nrows; ++i) {
        int64_t s0, s1;
        if (dp1) {
            s0 = m.dp1_star[r.rows[i]];
            s1 = s0 + 1;
        } else {
            s0 = m.star_ptr[r.rows[i]];
            s1 = m.star_ptr[r.rows[i] + 1];
        }
        bool any = false;
        for (int64_t s = s0; s < s1; ++s) {
            const int32_t a = m.star[s] >> 2;
            if (sc.slot[a] != sg) {
                sc.slot[a] = sg;
                sc.slot_of[a] = (int32_t)gptr.size() - 1;
                neighbours(m, a, nb);
                for (int32_t b : nb) {
                    bool touches;
                    if (dp1) {
                        touches = sc.col[b] == cg;
                    } else {
                        const int32_t *v = &m.tri[3 * (size_t)b];
                        touches = sc.col[v[0]] == cg || sc.col[v[1]] == cg || sc.col[v[2]] == cg;
                    }
                    if (touches && !(skip_same && a == b)) r.near_pairs.push_back({a, b, 0, 0, 0});
                }
                gptr.push_back((int32_t)r.near_pairs.size());
            }
            const int32_t slot = sc.slot_of[a];
            if (gptr[slot + 1] == gptr[slot]) continue;
            rs.push_back((slot << 2) | (m.star[s] & 3));
            any = true;
        }
        rptr.push_back((int32_t)rs.size());
        if (any) r.near_rows.push_back((int32_t)i);
    }
    r.near_slots = (int32_t)gptr.size() - 1;
    r.near_ints = std::move(gptr);
    r.near_ints.insert(r.near_ints.end(), rptr.begin(), rptr.end());
    r.near_ints.insert(r.near_ints.end(), rs.begin(), rs.end());
}

void clear_near(Request &r)
{
    r.near_pairs.clear();
    r.near_ints.clear();
    r.near_rows.clear();
    r.near_slots = 0;
}

int expand_near(Request &r)
{
    clear_near(r);
    if (r.near != BEM_NEAR_SINGULAR) return BEM_OK;
    if (r.space == BEM_P0)
        build_near_p0(r);
    else
        build_near_p1(r);
    return check_near_omega(r);
}

}  // namespace

int near_kind(const Request &r)
{
    const int g = r.op == BEM_LAPLACE_HYPS   ? 8
                : r.op == BEM_HELMHOLTZ_HYPS ? 9
                                             : kernel_op(r.op) + (r.space == BEM_P0 ? 0 : 4);
    return 2 * g + (r.prec == BEM_FP32 ? 1 : 0);
}

NearCount near_count(const Request &r)
{
    NearCount n;
    if (r.near_pairs.empty()) return n;
    n.reqs = 1;
    n.pairs = (int64_t)r.near_pairs.size();
    if (r.space != BEM_P0) {
        n.blocks = (int64_t)r.near_rows.size() * ((r.ncols + 255) / 256);
        n.ints = (int64_t)r.near_ints.size() + r.ncols;
    }
    return n;
}

NearLayout near_layout(int kind, const NearCount &n)
{
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const int g = kind >> 1;
    const bool p0 = g < 4, cplx = p0 ? g >= 2 : (g == 6 || g == 7 || g == 9);
    NearLayout L;
    L.pairs = al(sizeof(NearReq) * (size_t)n.reqs);
    L.blocks = al(L.pairs + sizeof(NearPair) * (size_t)n.pairs);
    L.ints = al(L.blocks + sizeof(NearBlock) * (size_t)n.blocks);
    L.staged = al(L.ints + sizeof(int32_t) * (size_t)n.ints);
    L.keys = L.staged;
    L.local = p0 ? L.keys : al(L.keys + sizeof(int4) * (size_t)n.pairs);
    L.bytes = p0 ? L.local : al(L.local + 9 * (cplx ? 2 : 1) * sizeof(double) * (size_t)n.pairs);
    return L;
}

void stage_near(const Request &r, const NearLayout &L, char *host, char *dev, char *out_dev, NearCount &at)
{
    const bem_mesh &m = *r.mesh;
    NearReq d{};
    d.xyz = m.d_xyz;
    d.g64 = m.d_g64;
    d.vtx = m.d_vtx;
    d.out = out_dev;
    d.k = is_complex_op(r.op) ? r.k : 0.0;
    d.ncols = (int32_t)r.ncols;
    d.transposed = is_adjoint_op(r.op) ? 1 : 0;
    d.dp1 = r.space == BEM_DP1 ? 1 : 0;
    NearPair *q = reinterpret_cast<NearPair *>(host + L.pairs) + at.pairs;
    for (size_t j = 0; j < r.near_pairs.size(); ++j) {
        q[j] = r.near_pairs[j];
        q[j].req = (int32_t)at.reqs;
    }
    const NearCount n = near_count(r);
    if (r.space != BEM_P0) {
        int32_t *h = reinterpret_cast<int32_t *>(host + L.ints) + at.ints;
        const int32_t *dv = reinterpret_cast<const int32_t *>(dev + L.ints) + at.ints;
        const size_t ng = (size_t)r.near_slots + 1;
        for (size_t j = 0; j < ng; ++j) h[j] = r.near_ints[j] + (int32_t)at.pairs;   // indices into the region
        std::memcpy(h + ng, r.near_ints.data() + ng, sizeof(int32_t) * (r.near_ints.size() - ng));
        std::memcpy(h + r.near_ints.size(), r.cols.data(), sizeof(int32_t) * (size_t)r.ncols);
        d.gptr = dv;
        d.rptr = dv + ng;
        d.rs = dv + ng + r.nrows + 1;
        d.cols = dv + r.near_ints.size();
        NearBlock *b = reinterpret_cast<NearBlock *>(host + L.blocks) + at.blocks;
        for (int32_t row : r.near_rows)
            for (int64_t c = 0; c < r.ncols; c += 256) *b++ = {(int32_t)at.reqs, row, (int32_t)c, 0};
    }
    reinterpret_cast<NearReq *>(host)[at.reqs] = d;
    at.reqs += n.reqs;
    at.pairs += n.pairs;
    at.blocks += n.blocks;
    at.ints += n.ints;
}

// Fixed triangles per workgroup of a P0 request: as many as leave 2,048
// workgroups, eight for each compute unit.  With half as many the units' shares
// differ by more than the tiles save, with twice as many the host's records do
// (701 x 3,001 by single triangles / tiles with 512, 2,048 and 4,096 workgroups,
// us: FP32 Helmholtz single layer, 4-point rule 54 / 49, 46, 48, 6-point 78 / 81,
// 75, 74; FP32 Laplace 52 / 29, 28, 33; FP64 Helmholtz double layer, 6-point
// 152 / 164, 149, 145).  Below that the single triangles fill the chip better
// (512 x 1,024 with the 6-point rule: alike from 512 workgroups on).
static int32_t p0_tile(int64_t nfix, int64_t nchunk)
{
    int32_t tile = kTileP0;
    while (tile > 1 && (nfix + tile - 1) / tile * nchunk < 2048) tile /= 2;
    return tile;
}

size_t plain_workspace(const Request &r, size_t limit)
{
    const bem_mesh &m = *r.mesh;
    const std::vector<int32_t> &fix = r.fixrows ? r.rows : r.cols, &lane = r.fixrows ? r.cols : r.rows;
    const size_t nf = fix.size(), nl = lane.size();
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    auto bytes = [&](size_t chunks, size_t ints) {
        return al(sizeof(ReqDev)) + al(sizeof(EntryBlock) * nf * chunks) + al(16 * chunks + 4 * ints) + al(8);
    };
    if (r.space == BEM_P0) return bytes((nl + kBlockLanes - 1) / kBlockLanes, nl);
    // every chunk but the last lacks room for one more star
    size_t stars = nl;
    if (r.space == BEM_P1) {
        stars = 0;
        for (int32_t d : lane) stars += (size_t)(m.star_ptr[d + 1] - m.star_ptr[d]);
    }
    const size_t least = r.space == BEM_P1 ? (size_t)std::max<int64_t>(1, kBlockLanes - m.max_star) : kBlockLanes - 1;
    const size_t most = bytes(std::min(nl, stars / least + 1), 2 * stars + 2 * nl + 1);
    if (most <= limit) return most;
    LaneSet ls;
    build_lane_set(m, r.space, lane.data(), (int64_t)nl, ls, true);
    return bytes((size_t)ls.nchunk(), ls.ints() - ls.chunk.size());
}

bool row_touches(const Request &r)
{
    // the dofs with a triangle that shares a vertex with one of the fixed
    // stars', few for few fixed dofs, are looked up among the lane dofs
    const bem_mesh &m = *r.mesh;
    std::vector<int32_t> v, touch;
    auto unique = [](std::vector<int32_t> &x) {
        std::sort(x.begin(), x.end());
        x.erase(std::unique(x.begin(), x.end()), x.end());
    };
    for (size_t f = 0; 2 * f + 1 < r.fix.size(); ++f)
        for (int32_t s = r.fix[2 * f]; s < r.fix[2 * f + 1]; ++s)
            for (int a = 0; a < 3; ++a) v.push_back(m.tri[3 * (size_t)(m.star[s] >> 2) + a]);
    unique(v);
    for (int32_t u : v)
        for (int64_t s = m.star_ptr[u]; s < m.star_ptr[u + 1]; ++s)
            for (int a = 0; a < 3; ++a) {
                const int64_t t = m.star[s] >> 2;
                touch.push_back(r.space == BEM_P1 ? m.tri[3 * t + a] : (int32_t)(3 * t + a));
            }
    unique(touch);
    for (int32_t d : r.fixrows ? r.cols : r.rows)
        if (std::binary_search(touch.begin(), touch.end(), d)) return true;
    return false;
}

int expand_request(Request &r, const PairRoom &room)
{
    const bem_mesh &m = *r.mesh;
    if (r.op < 0 || r.op > 7) return fail(BEM_E_ARG, "unknown operator");
    if (r.space != BEM_P0 && r.space != BEM_P1 && r.space != BEM_DP1) return fail(BEM_E_ARG, "unknown space");
    if ((r.op == BEM_LAPLACE_HYPS || r.op == BEM_HELMHOLTZ_HYPS) && r.space != BEM_P1)
        return fail(BEM_E_ARG, "the hypersingular operator needs continuous (P1) functions");
    if (r.prec != BEM_FP32 && r.prec != BEM_FP64) return fail(BEM_E_ARG, "unknown precision");
    if (r.near != BEM_NEAR_ERROR && r.near != BEM_NEAR_SKIP && r.near != BEM_NEAR_SINGULAR)
        return fail(BEM_E_ARG, "unknown near-field policy");
    if (is_complex_op(r.op)) {
        if (!(std::isfinite(r.k) && r.k > 0.0)) return fail(BEM_E_ARG, "Helmholtz needs a finite wavenumber k > 0");
    } else if (r.k != 0.0) {
        return fail(BEM_E_ARG, "Laplace needs k = 0");
    }
    const int64_t ndof = space_ndof(m, r.space);
    for (int32_t v : r.rows)
        if (v < 0 || v >= ndof) return fail(BEM_E_ARG, "row index out of range");
    for (int32_t v : r.cols)
        if (v < 0 || v >= ndof) return fail(BEM_E_ARG, "column index out of range");
    if (r.nrows > INT32_MAX || r.ncols > INT32_MAX) return fail(BEM_E_ARG, "request dimension too large");

    r.ext = nullptr;
    // the smaller side is fixed; an adjoint double layer is evaluated as the
    // double layer with test and trial exchanged (Eqs. dlp, adlp:
    // [K'_h]_ij = [K_h]_ji for the same space on both sides)
    r.fixrows = r.ncols >= r.nrows ? 1 : 0;
    r.rowfix = is_adjoint_op(r.op) ? 1 - r.fixrows : r.fixrows;
    const std::vector<int32_t> &fix_dofs = r.fixrows ? r.rows : r.cols;
    const std::vector<int32_t> &lane_dofs = r.fixrows ? r.cols : r.rows;
    r.row = row_pays(r, (int64_t)fix_dofs.size());
    r.paired = !r.row && !r.plain && room.budget > 0 && pairs_pay(r, fix_dofs, lane_dofs, room);
    if (r.paired) {
        plan_pairs(m, r.space, kernel_op(r.op), r.prec, r.rowfix != 0, fix_dofs.data(), (int64_t)fix_dofs.size(),
                   lane_dofs.data(), (int64_t)lane_dofs.size(), room.budget, r.pairs);
        r.pair_error = r.near == BEM_NEAR_ERROR && pairs_touch(m, r.pairs);
        r.nfix = r.nlane = r.nchunk = r.nblocks = 0;   // no block table
        r.elem_bytes = out_elem_bytes(r.op, r.prec);
        r.evals = r.pairs.pairs * m.q * m.q;
        r.in_bytes = align16(4 * r.pairs.ints.size());
        r.out_bytes = align16((size_t)r.entries() * r.elem_bytes);
        const int rc = expand_near(r);
        r.batch_bytes = request_bytes(r);
        return rc;
    }
    expand_fixed(m, r.space, fix_dofs.data(), (int64_t)fix_dofs.size(), r);
    if (r.row)
        build_row_set(m, r.space, r.nfix, lane_dofs.data(), (int64_t)lane_dofs.size(), r.own, r.row_split);
    else
        build_lane_set(m, r.space, lane_dofs.data(), (int64_t)lane_dofs.size(), r.own, true);
    r.nlane = (int64_t)r.own.lane.size();
    r.nchunk = r.own.nchunk();
    r.ndistinct = r.own.ndistinct;
    r.tile = r.space == BEM_P0 ? p0_tile(r.nfix, r.nchunk) : 1;
    const int rc = expand_near(r);
    if (rc != BEM_OK) return rc;
    finalize_sizes(r);
    return BEM_OK;
}

void expand_single_fixed(Request &r, int32_t dof, int rowfix, const LaneRef *ext)
{
    clear_near(r);
    r.ext = ext;
    r.row = false;
    r.tile = 1;
    r.fixrows = rowfix;
    r.rowfix = is_adjoint_op(r.op) ? 1 - rowfix : rowfix;
    r.own.lane.clear();
    r.own.chunk.clear();
    r.own.seg_ptr.clear();
    r.own.seg.clear();
    r.own.pos.clear();
    expand_fixed(*r.mesh, r.space, &dof, 1, r);
    r.nlane = ext->nlane;
    r.nchunk = ext->nchunk;
    r.ndistinct = ext->ndistinct;
    if (r.fixrows) {
        r.nrows = 1;
        r.ncols = ext->ndof;
    } else {
        r.nrows = ext->ndof;
        r.ncols = 1;
    }
    finalize_sizes(r);
}

size_t request_bytes(const Request &r)
{
    // descriptor, inputs, status, outputs, block table, launch-timing records.  By
    // triangle pairs the device's part is the larger: the entries lie there once
    // more than in the staging, behind the local matrices, not in both of one sum.
    return sizeof(ReqDev) + r.in_bytes + 8 + r.out_bytes + (size_t)r.nblocks * (sizeof(EntryBlock) + 16) +
           (r.near_pairs.empty() ? 0 : near_layout(near_kind(r), near_count(r)).bytes) +
           (r.paired ? r.pairs.work + 512 : 0) + 512;
}

void describe_request(const Request &r, ReqDev &d)
{
    const bem_mesh &m = *r.mesh;
    d.g32 = m.d_g32;
    d.g64 = m.d_g64;
    d.vtx = m.d_vtx;
    if (r.ext) {
        d.lane = r.ext->lane;
        d.seg_ptr = r.ext->seg_ptr;
        d.seg = r.ext->seg;
    } else {
        d.lane = d.seg_ptr = d.seg = nullptr;
    }
    d.lpos = nullptr;
    d.sptr = r.space == BEM_P1 ? m.d_sptr : nullptr;
    d.group = r.space == BEM_P1 ? 3 : 0;
    d.split = r.row_split;
    d.fstar = m.d_star;
    if (r.fixrows) {   // output position of (fixed f, lane-side dof d): out[f * sf + d * sl]
        d.sf = r.ncols;
        d.sl = 1;
    } else {
        d.sf = 1;
        d.sl = r.ncols;
    }
    d.nrows = (int32_t)r.nrows;
    d.ncols = (int32_t)r.ncols;
    d.rowfix = r.rowfix;
    d.near_error = r.near == BEM_NEAR_ERROR ? 1 : 0;
    d.k = r.k;
    d.kk = r.k / (2.0 * 3.14159265358979323846);
    d.kl = wave_low(r.k, d.kk);
    d.kend = wave_end(d.kk, kernel_op(r.op));
    d.out = nullptr;
    d.status = nullptr;
}

size_t stage_own_inputs(const Request &r, char *host_base, char *dev_base, size_t off, ReqDev &d)
{
    if (r.ext) return r.in_bytes;
    char *h = host_base + off;
    char *dv = dev_base + off;
    auto put = [&](const std::vector<int32_t> &v) -> const int32_t * {
        if (v.empty()) return nullptr;
        std::memcpy(h, v.data(), 4 * v.size());
        const int32_t *dp = reinterpret_cast<const int32_t *>(dv);
        h += 4 * v.size();
        dv += 4 * v.size();
        return dp;
    };
    d.lane = put(r.own.lane);
    d.seg_ptr = put(r.own.seg_ptr);
    d.seg = put(r.own.seg);
    d.lpos = put(r.own.pos);
    if (r.tile > 1) d.sptr = put(r.fix);
    return r.in_bytes;
}

size_t stage_request_inputs(Request &r, char *host_base, char *dev_base, size_t off, ReqDev &d)
{
    describe_request(r, d);
    return stage_own_inputs(r, host_base, dev_base, off, d);
}

void finish_descriptor(const Request &r, char *dev_base, size_t off_out, size_t off_status, ReqDev &d)
{
    (void)r;
    d.out = dev_base + off_out;
    d.status = reinterpret_cast<int32_t *>(dev_base + off_status);
}

int64_t write_blocks(const Request &r, int32_t ri, EntryBlock *out)
{
    const bem_mesh &m = *r.mesh;
    const int32_t *ch = r.ext ? r.ext->chunk_host : r.own.chunk.data();
    const float *lgeo = r.ext ? r.ext->geo : nullptr;
    const int4 *lmeta = r.ext ? r.ext->meta : nullptr;
    int64_t n = 0;
    for (int32_t f = 0; f < (int32_t)r.nfix; f += r.tile) {
        int32_t s0, s1;
        if (r.tile > 1) {   // positions in the list of fixed triangles
            s0 = f;
            s1 = std::min((int32_t)r.nfix, f + r.tile);
        } else if (r.space == BEM_P0) {
            s0 = r.fix[f];
            s1 = s0 + 1;
        } else {
            s0 = r.fix[2 * f];
            s1 = r.fix[2 * f + 1];
        }
        for (int32_t c = 0; c < (int32_t)r.nchunk; ++c) {
            EntryBlock &b = out[n++];
            b.req = (ri << 1) | (r.rowfix ? 1 : 0);
            b.fixed = f;
            b.s0 = s0;
            b.s1 = s1;
            b.chunk = make_int4(ch[4 * c], ch[4 * c + 1], ch[4 * c + 2], ch[4 * c + 3]);
            b.lgeo = lgeo;
            b.lmeta = r.separated ? nullptr : lmeta;
            // the fixed side's records: P1 star records per star entry, P0
            // the mesh's triangle records
            b.sgeo = r.space != BEM_P0 ? m.d_sgeo : m.d_g32;
            b.smeta = r.space != BEM_P0 ? m.d_smeta : m.d_vtx;
        }
    }
    return n;
}

int request_key(const Request &r)
{
    return ((((r.row || r.tile > 1 ? 8 : 0) + kernel_op(r.op)) * 2 + kernel_space(r.space)) * 2 + r.prec) * 2 +
           (r.mesh->q == 6 ? 1 : 0);
}

void prebuild_staging(Request &r)
{
    r.key = request_key(r);
    r.pre_blocks.resize((size_t)r.nblocks);
    write_blocks(r, 0, r.pre_blocks.data());
    describe_request(r, r.pre_dev);
}

}  // namespace bem

// ---------------------------------------------------------------------------
// Mesh creation / destruction.
using namespace bem;

namespace bem {
int mesh_create_impl(const double *xyz, int64_t nv, const int32_t *tri, int64_t nt, int q, bem_mesh **out)
{
    if (!xyz || !tri || !out) return fail(BEM_E_ARG, "null pointer");
    if (nv < 3 || nt < 1) return fail(BEM_E_ARG, "mesh needs at least 3 vertices and 1 triangle");
    if (q != 4 && q != 6) return fail(BEM_E_ARG, "quad_points must be 4 or 6");
    if (nt > (INT32_MAX >> 2) || nv > INT32_MAX) return fail(BEM_E_ARG, "mesh too large for 32-bit indices");
    for (int64_t i = 0; i < 3 * nv; ++i)
        if (!std::isfinite(xyz[i])) return fail(BEM_E_ARG, "non-finite vertex coordinate");
    for (int64_t i = 0; i < 3 * nt; ++i)
        if (tri[i] < 0 || tri[i] >= nv) return fail(BEM_E_ARG, "triangle vertex index out of range");
    for (int64_t t = 0; t < nt; ++t)
        if (tri[3 * t] == tri[3 * t + 1] || tri[3 * t] == tri[3 * t + 2] || tri[3 * t + 1] == tri[3 * t + 2])
            return fail(BEM_E_ARG, "triangle with a repeated vertex");

    bem_mesh *m = new (std::nothrow) bem_mesh();
    if (!m) return fail(BEM_E_OOM, "host allocation failed");
    m->nv = nv;
    m->nt = nt;
    m->q = q;
    m->xyz.assign(xyz, xyz + 3 * nv);
    m->tri.assign(tri, tri + 3 * nt);
    m->star_ptr.assign(nv + 1, 0);
    for (int64_t i = 0; i < 3 * nt; ++i) m->star_ptr[tri[i] + 1]++;
    for (int64_t v = 0; v < nv; ++v) m->star_ptr[v + 1] += m->star_ptr[v];
    m->star.resize(3 * nt);
    {
        std::vector<int64_t> fill(m->star_ptr.begin(), m->star_ptr.end() - 1);
        for (int64_t t = 0; t < nt; ++t)
            for (int k = 0; k < 3; ++k) m->star[fill[tri[3 * t + k]]++] = (int32_t)((t << 2) | k);
    }
    m->dp1_star.resize(3 * nt);
    for (int64_t s = 0; s < 3 * nt; ++s) m->dp1_star[3 * (size_t)(m->star[s] >> 2) + (m->star[s] & 3)] = (int32_t)s;
    for (int64_t v = 0; v < nv; ++v) m->max_star = std::max<int>(m->max_star, (int)(m->star_ptr[v + 1] - m->star_ptr[v]));
    if (m->max_star > kBlockLanes) {
        delete m;
        return fail(BEM_E_ARG, "a vertex belongs to more than 256 triangles");
    }
    double sj = 0.0, se = 0.0;
    for (int64_t t = 0; t < nt; ++t) {
        const double *a = &xyz[3 * tri[3 * t]], *b = &xyz[3 * tri[3 * t + 1]], *c = &xyz[3 * tri[3 * t + 2]];
        double e1[3], e2[3];
        for (int d = 0; d < 3; ++d) {
            e1[d] = b[d] - a[d];
            e2[d] = c[d] - a[d];
        }
        const double N[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2], e1[0] * e2[1] - e1[1] * e2[0]};
        sj += std::sqrt(N[0] * N[0] + N[1] * N[1] + N[2] * N[2]);
        double e3[3] = {c[0] - b[0], c[1] - b[1], c[2] - b[2]};
        const double l1 = std::sqrt(e1[0] * e1[0] + e1[1] * e1[1] + e1[2] * e1[2]),
                     l2 = std::sqrt(e2[0] * e2[0] + e2[1] * e2[1] + e2[2] * e2[2]),
                     l3 = std::sqrt(e3[0] * e3[0] + e3[1] * e3[1] + e3[2] * e3[2]);
        se += l1 + l2 + l3;
        m->max_edge = std::max(m->max_edge, std::max(l1, std::max(l2, l3)));
    }
    m->mean_J = sj / nt;
    m->mean_edge = se / (3.0 * nt);
    for (int d = 0; d < 3; ++d) {
        double lo = INFINITY, hi = -INFINITY;
        for (int64_t v = 0; v < nv; ++v) {
            lo = std::min(lo, xyz[3 * v + d]);
            hi = std::max(hi, xyz[3 * v + d]);
        }
        m->box_lo[d] = lo;
        m->box_inv[d] = hi > lo ? 1.0 / (hi - lo) : 0.0;
    }

    hipError_t e = hipGetDevice(&m->device);
    int32_t *d_tri = nullptr, *d_bad = nullptr;
    const size_t b32 = sizeof(float) * kGeo32Stride * nt, b64 = sizeof(double) * kGeo64Stride * nt,
                 bv = sizeof(int4) * nt;
    int rc = BEM_OK;
    int32_t bad = 0;
    if (e == hipSuccess) e = alloc_device((void **)&m->d_g32, b32);
    if (e == hipSuccess) e = alloc_device((void **)&m->d_g64, b64);
    if (e == hipSuccess) e = alloc_device((void **)&m->d_vtx, bv);
    // what the host has: vertices, star entries, triangles, star ranges and,
    // after them, the degenerate flag; one allocation
    const int64_t ns = 3 * nt;
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t o_star = al(sizeof(double) * 3 * nv), o_tri = al(o_star + sizeof(int32_t) * ns),
                 o_sptr = al(o_tri + sizeof(int32_t) * 3 * nt), bh = al(o_sptr + sizeof(int32_t) * (nv + 2));
    if (e == hipSuccess) e = alloc_device((void **)&m->d_xyz, bh);
    if (e == hipSuccess) {
        char *base = reinterpret_cast<char *>(m->d_xyz);
        m->d_star = reinterpret_cast<int32_t *>(base + o_star);
        d_tri = reinterpret_cast<int32_t *>(base + o_tri);
        m->d_sptr = reinterpret_cast<int32_t *>(base + o_sptr);
        d_bad = m->d_sptr + nv + 1;
        std::vector<int32_t> sp(m->star_ptr.begin(), m->star_ptr.end());
        sp.push_back(0);
        e = hipMemcpy(m->d_xyz, xyz, sizeof(double) * 3 * nv, hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipMemcpy(m->d_star, m->star.data(), sizeof(int32_t) * ns, hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipMemcpy(d_tri, tri, sizeof(int32_t) * 3 * nt, hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipMemcpy(m->d_sptr, sp.data(), sizeof(int32_t) * (nv + 2), hipMemcpyHostToDevice);
    }
    if (e == hipSuccess) e = launch_geometry(m->d_xyz, d_tri, nt, q, m->d_g32, m->d_g64, m->d_vtx, d_bad, 0);
    if (e == hipSuccess) e = hipMemcpy(&bad, d_bad, sizeof(int32_t), hipMemcpyDeviceToHost);
    // star tables: the packed star entries and, per entry, its triangle's
    // FP32 record and vertex ids with the local vertex in w
    if (e == hipSuccess) e = alloc_device((void **)&m->d_sgeo, sizeof(float) * kGeo32Stride * ns);
    if (e == hipSuccess) e = alloc_device((void **)&m->d_smeta, sizeof(int4) * ns);
    if (e == hipSuccess) e = launch_gather(m->d_g32, m->d_vtx, m->d_star, 2, ns, m->d_sgeo, m->d_smeta, 0);
    if (e == hipSuccess) e = hipStreamSynchronize(0);
    if (e != hipSuccess)
        rc = fail(e == hipErrorOutOfMemory ? BEM_E_OOM : BEM_E_DEVICE, std::string("mesh upload: ") + hipGetErrorString(e));
    else if (bad)
        rc = fail(BEM_E_ARG, "degenerate triangle (zero area)");
    if (rc != BEM_OK) {
        for (void *p : {(void *)m->d_g32, (void *)m->d_g64, (void *)m->d_vtx, (void *)m->d_sgeo, (void *)m->d_smeta,
                        (void *)m->d_xyz})
            if (p) (void)hipFree(p);
        delete m;
        return rc;
    }
    m->dev_bytes = b32 + b64 + bv + bh + 3 * (size_t)nt * (4 * kGeo32Stride + sizeof(int4));
    *out = m;
    return BEM_OK;
}

int mesh_destroy_impl(bem_mesh *m)
{
    if (!m) return fail(BEM_E_ARG, "null mesh");
    if (m->inflight.load() != 0) return fail(BEM_E_BUSY, "requests on this mesh are still in flight");
    for (void *p : {(void *)m->d_g32, (void *)m->d_g64, (void *)m->d_vtx, (void *)m->d_sgeo, (void *)m->d_smeta,
                    (void *)m->d_xyz})
        (void)hipFree(p);
    delete m;
    return BEM_OK;
}
}  // namespace bem
