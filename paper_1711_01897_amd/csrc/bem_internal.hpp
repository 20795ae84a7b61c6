// Internal declarations of libbem (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <condition_variable>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "bem.h"

namespace bem {

struct Request;

// ---------------------------------------------------------------------------
// Device layout of one triangle.
//
// FP32 record, 16 floats (64 B, one load of four float4), for the
// compensated FP32 path:
//   [0..2]   centroid, high part (float of the FP64 centroid)   [3]  J = |(b-a)x(c-a)|
//   [4..6]   centroid, low part  (float of the FP64 remainder)  [7]  n_x
//   [8..10]  e1 = b - a                                         [11] n_y
//   [12..14] e2 = c - a                                         [15] n_z
// (n the unit normal).  Kernels expand it in registers to the working
// layout of n32<Q>() words: [0..2] centroid high, [3] J, [4..6] centroid
// low, [8..10] n, and from [12] the quadrature points relative to the
// centroid, x_p - c = (xi_p - 1/3) e1 + (eta_p - 1/3) e2, point-major.
// Differences of two triangles' positions are formed as (hi_a - hi_b) +
// (lo_a - lo_b) + (offset_p - offset_q): the large centroid parts cancel
// first, so the result keeps FP32 relative accuracy in |x - y| wherever the
// mesh sits in space.
//
// FP64 record, 24 doubles (192 B), for the plain FP64 path:
//   [0..2] unit normal  [3] J  [4..] absolute quadrature points, point-major.
constexpr int kGeo32Stride = 16;
constexpr int kGeo64Stride = 24;
constexpr int kBlockLanes = 256;    // lane-side items per workgroup (4 wavefronts)
constexpr int kTileP0 = 8;          // P0: fixed triangles per workgroup at most
constexpr int kStage = 8;           // fixed-side triangles staged in LDS at a time

// One request as the entry kernels see it.
//
// "fixed" side: one triangle (P0) or one vertex star (P1) shared by the
// lanes of a workgroup; "lane" side: one triangle per lane, grouped in
// chunks of at most kBlockLanes lanes.  rowfix = 1 means the fixed side is
// the test (row) side.  Output position (fixed f, lane-side dof d) is
// out[f * sf + d * sl].
struct ReqDev {
    const float *g32;
    const double *g64;
    const int4 *vtx;           // vertex ids per triangle (x, y, z; w unused)
    const int32_t *fstar;      // P1: the mesh star table (packed triangle << 2 | local vertex); block
                               // records name the fixed dof's entries [s0, s1)
    const int32_t *lane;       // triangle per lane position
    const int32_t *seg_ptr;    // P1: per lane-side dof, range into seg
    const int32_t *seg;        // P1: packed (lane slot within the chunk << 2 | local vertex)
    const int32_t *lpos;       // P1: output position of each lane-side dof (null: its own index)
    const int32_t *sptr;       // row form: the mesh's star ranges per vertex (null: `lane` holds star entries);
                               // P0 tiles: the fixed triangles
    int32_t group, split;      // row form: log2 of the threads per lane dof, and of the shares of a fixed star
    void *out;                 // final output, row-major nrows x ncols
    int32_t *status;           // set to 1: a vertex-sharing pair was met under BEM_NEAR_ERROR
    int64_t sf, sl;
    int32_t nrows, ncols;
    int32_t rowfix;
    int32_t near_error;
    double k;                  // wavenumber
    double kk;                 // k / (2 pi): phase in turns per unit length
    double kl;                 // k / pi - 2 kk: what the FP64 phase adds to 2 kk (wave_low)
    double kend;               // where the FP64 phase ends (wave_end)
};

// k / pi minus its rounded value 2 kk, from 64-bit mantissas.
inline double wave_low(double k, double kk)
{
    return (double)((long double)k / 3.14159265358979323846264338327950288L - 2.0L * (long double)kk);
}

// The distance of 2^50 half turns (double layer), or its square (else).
inline double wave_end(double kk, int kernel_op)
{
    const double r = 0x1p49 / kk;
    return kernel_op == BEM_HELMHOLTZ_DLP ? r : r * r;
}

struct EntryBlock {  // one workgroup of entry work (64 bytes, read with one scalar load)
    int32_t req;           // (request index << 1) | 1 if the test side is fixed (row request): the kernel
                           // picks its code path before the request descriptor arrives
    int32_t fixed;         // fixed position
    int32_t s0, s1;        // P1: the fixed dof's star, entries [s0, s1) of the mesh star table; P0: s0 = the fixed triangle
    int4 chunk;            // lane side: first lane, lanes, first dof, dofs
    const float *lgeo;     // lane records gathered per lane position (or null: gather through R.lane)
    const int4 *lmeta;     // their vertex ids; null with lgeo set: the sides are separated (no vertex-sharing
                           // pair can occur, the kernels skip the test)
    const float *sgeo;     // P1: the mesh's star records (FP32), indexed by star entry; P0: its triangle records
    const int4 *smeta;     // their vertex ids (P1: w = local vertex of the star's dof)
};

// Kernel variant: one compiled instantiation of the entry kernel (it serves
// both fixed sides).
struct Variant {
    int op, space, prec, q;
    int row = 0;       // P1: the row form; P0: tiles (counted with the other form in the statistics)
    int persist = 0;   // statistics only: the resident (persistent) form of the kernel
    bool operator<(const Variant &o) const {
        if (op != o.op) return op < o.op;
        if (space != o.space) return space < o.space;
        if (prec != o.prec) return prec < o.prec;
        if (q != o.q) return q < o.q;
        return persist < o.persist;
    }
};

// Block table of a request, written by the host: request index `ri` inside
// its batch, blocks in (fixed, chunk) order; returns the count.
int64_t write_blocks(const Request &r, int32_t ri, EntryBlock *out);

// Launchers (entries.hip).  Return hipSuccess or the launch error.
// tclock (optional, device memory, 2 * nblocks entries): receives each
// workgroup's start and end on the device's constant-rate clock.
// start/stop (optional): HIP events recorded around the launch on its stream.
hipError_t launch_entries(const Variant &v, const ReqDev *reqs, const EntryBlock *blocks, int64_t nblocks, hipStream_t s,
                          unsigned long long *tclock = nullptr, hipEvent_t start = nullptr, hipEvent_t stop = nullptr);

// ---------------------------------------------------------------------------
// Persistent service of batches.
//
// One launch of the entry kernel stays resident and serves a stream of
// batches of one kernel variant.  The host publishes each batch (its
// descriptors and block records already in host-coherent staging) as an
// entry of a ring in host-coherent memory, in sequence order.  Workgroup 0
// watches the ring (one thread) and copies each published entry to device
// memory together with its claim word; the other workgroups claim blocks
// with atomic adds on the claim words, oldest batch first, and run the same
// per-block code as the launched kernels.  Any workgroup can claim any
// block, so a launch never depends on all of its workgroups being resident.
// The workgroup that ends a batch's last block stores seq + 1 into the
// batch's completion word in host memory.  The launch ends when the host asks
// it to or no entry has been published for a given number of device-clock
// ticks: the watching thread stores the first sequence number it did not
// take into the exit word, and every waiting workgroup returns.  The host
// publishes entry i again only after the batch it last held has completed.
constexpr int kPersistRing = 64;    // ring entries (more than batches in flight)

struct PersistEntry {               // host-coherent; seq1 written last
    const ReqDev *reqs;
    const EntryBlock *blocks;
    unsigned long long *clock;      // per block {start, end} device clock, or null
    int64_t nblk;
    uint64_t seq1;                  // sequence number + 1 once published
    uint64_t pad[3];
};
static_assert(sizeof(PersistEntry) == 64, "ring entries are 64 bytes");

struct PersistHost {                // host-coherent words shared by the persistent launches
    PersistEntry ring[kPersistRing];
    uint64_t done[kPersistRing][8];   // done[i][0] = seq + 1 of the last batch of ring entry i completed
    uint64_t stop;                    // the host asks launches with id <= stop to end
    uint64_t pad0[7];
    uint64_t exit_word;               // id << 40 | (first sequence number not taken + 1), stored by a
                                      // launch as it ends
    uint64_t pad1[7];
};

struct PersistItem {                // a published batch as the workers read it (device memory)
    const ReqDev *reqs;
    const EntryBlock *blocks;
    unsigned long long *clock;
    int64_t nblk;
    uint64_t pad[4];
};

// Claim word of ring entry i: (seq mod 2^16) << 48 | nblk << 32 | blocks
// claimed, seq the batch the entry holds.  An atomic add of one claims
// block "blocks claimed" when that is below nblk; the tag names the batch
// the claim belongs to whatever batch the claimer expected (a workgroup's
// cursor is never 2^15 batches away from the batches an entry can hold), so
// no claim is lost when an entry is reused.
struct PersistCtl {                 // device memory, reset before each launch
    unsigned long long cur;         // every batch before cur has no unclaimed block
    unsigned long long pad0[15];
    unsigned int stop;              // the watcher has left: waiting workgroups return
    unsigned int pad1[31];
    PersistItem item[kPersistRing];
    unsigned long long claim[kPersistRing][16];   // one 128-byte line each
    unsigned int done[kPersistRing][32];          // blocks finished, one line each
};
constexpr int kPersistMaxBlocks = 65535;   // per batch (the claim word's nblk field)

struct PersistArgs {
    const PersistHost *host;        // device address of the host words
    uint64_t *done;                 // device address of host->done
    uint64_t *exit_word;            // device address of host->exit_word
    PersistCtl *ctl;
    uint64_t seq0;                  // first sequence number this launch serves
    uint64_t id;                    // launch number: the launch ends once host->stop >= id
    long long idle_ticks;           // device-clock ticks without a new entry before the launch ends
};

// Enqueues the reset of a.ctl for a launch that starts at sequence number
// a.seq0, then the persistent launch of variant v with `groups` workgroups
// (workgroup 0 watches the ring); start/stop events (optional) around the
// persistent launch.
hipError_t launch_persistent(const Variant &v, const PersistArgs &a, int groups, hipStream_t s,
                             hipEvent_t start = nullptr, hipEvent_t stop = nullptr);
// Resident workgroups per compute unit of the persistent kernel of variant v
// (0 if there is none).
int persistent_occupancy(const Variant &v);

hipError_t launch_geometry(const double *xyz, const int32_t *tri, int64_t nt, int q, float *g32, double *g64,
                           int4 *vtx, int32_t *bad, hipStream_t s);
// geo[i] = FP32 record of triangle index[i] >> shift, meta[i] = its vertex
// ids (w = index[i] & 3 when shift == 2, else 0); i < n.
hipError_t launch_gather(const float *g32, const int4 *vtx, const int32_t *index, int shift, int64_t n, float *geo,
                         int4 *meta, hipStream_t s);
// ---------------------------------------------------------------------------
// Vertex-sharing (singular) triangle pairs of BEM_NEAR_SINGULAR requests
// (near.hip).  The host lists the pairs by triangle index; the device finds
// the shared vertices, integrates each pair (one workgroup) and, for P1 and
// DP1, adds the pairs' 3 x 3 local matrices to the entries (one thread per
// entry of a row that has any).  The requests of a batch with one operator,
// space and precision share a region: staged part (copied to the device) |
// what the kernels write for each other.
struct NearPair {
    int32_t a, b;              // row-side and column-side triangle
    int32_t req, pad;          // request within the region
    int64_t entry;             // P0: the entry's position in the output
};
static_assert(sizeof(NearPair) == 24, "near pairs are 24 bytes");

struct NearReq {
    const double *xyz;         // mesh: vertices, FP64 records, vertex ids per triangle
    const double *g64;
    const int4 *vtx;
    void *out;
    // P1 and DP1: pairs [gptr[s], gptr[s + 1]) of the region belong to the
    // request's row-side triangle s; row r's star is rs[rptr[r] .. rptr[r + 1])
    // (triangle s << 2 | local vertex); cols: the column dofs
    const int32_t *gptr, *rptr, *rs, *cols;
    double k;                  // wavenumber
    int32_t ncols;
    int32_t transposed;        // the kernel's test triangle is the column's (adjoint double layer)
    int32_t dp1, pad;
};

struct NearBlock {             // P1: up to 256 columns of one row
    int32_t req, row, col0, pad;
};

struct NearCount {             // sizes of a region, or the part of it that precedes a request
    int64_t reqs = 0, pairs = 0, blocks = 0, ints = 0;
};

struct NearLayout {
    size_t pairs, blocks, ints, staged;   // the requests' descriptors come first; `staged` bytes are copied
    size_t keys, local, bytes;            // written on the device: column dofs per pair, local matrices
};

// Region kind of a request: 2 g + fp32, g = 0..3 the P0 kernel operators, 4 + (0..3) the P1 ones, 8 and 9 the
// Laplace and Helmholtz hypersingular operators.
constexpr int kNearKinds = 20;
int near_kind(const Request &r);
NearCount near_count(const Request &r);
NearLayout near_layout(int kind, const NearCount &n);
// Writes request r's part of a region's staged image at host (dev: the
// region's device address, out_dev: r's output on the device); `at` is
// advanced past it.
void stage_near(const Request &r, const NearLayout &L, char *host, char *dev, char *out_dev, NearCount &at);
// Enqueues the kernels of a staged region.
hipError_t launch_near(int kind, const NearLayout &L, const NearCount &n, char *dev, hipStream_t s);

// Copies bytes (a multiple of 16, both addresses 16-byte aligned) from src
// (device-visible host staging) to dst (device) with a kernel on stream s.
hipError_t launch_stage_copy(const void *src, void *dst, size_t bytes, hipStream_t s);

// ---------------------------------------------------------------------------
// P1 and DP1 blocks by triangle pairs (dense.cpp; kernels in entries.hip): both
// sides' dofs along a Morton curve, cut into panels of whole stars, a panel
// being the distinct triangles of its dofs' stars and, per dof, its star as
// (index into them << 2 | local vertex) and its output position.  A panel of
// the fixed side against one of the lane side is one launch of local matrices
// into a workspace and one that adds them to the entries; an entry's sum does
// not depend on where the cuts are.
struct PairPanel {
    int32_t ntri = 0, ndof = 0;
    size_t tri = 0, ptr = 0, src = 0, pos = 0;   // places in PairPlan::ints
};
struct PairPlan {
    std::vector<int32_t> ints;
    std::vector<PairPanel> fix, lane;
    size_t work = 0;        // workspace bytes of the largest pair of panels
    int64_t pairs = 0;      // triangle pairs over all panels
    int op = 0, prec = 0;
    bool ltrial = true;     // the lane side is the trial side
};
// Plan of fix x lane with at most `budget` bytes of workspace.  entries_panelled:
// the caller holds the entries of a panel of the fixed side in buffers of its own.
void plan_pairs(const bem_mesh &m, int space, int op, int prec, bool ltrial, const int32_t *fix, int64_t nfix,
                const int32_t *lane, int64_t nlane, size_t budget, PairPlan &P, bool entries_panelled = false);
// Whether two of the plan's triangles, one of each side, share a vertex.
bool pairs_touch(const bem_mesh &m, const PairPlan &P);
// What a request by triangle pairs may use: workspace bytes (0: it may not be),
// and whether its entries go to host memory (a served request).
struct PairRoom {
    size_t budget = 0;
    bool served = false;
};
// Whether a request is worth it (see the rule at its definition).
bool pairs_pay(const Request &r, const std::vector<int32_t> &fix, const std::vector<int32_t> &lane, const PairRoom &room);
// Enqueues one pair of panels: ints (device copy of P.ints), work (P.work bytes), entries at
// out[fixed position * sf + lane position * sl], the fixed position being the dof's in the caller's list
// or, with in_panel, in the panel.
hipError_t launch_pairs(const bem_mesh &m, const PairPlan &P, const PairPanel &f, const PairPanel &l, const int32_t *ints,
                        void *work, void *out, int64_t sf, int64_t sl, double k, hipStream_t s, bool in_panel = false,
                        hipEvent_t between = nullptr);
// Workgroups of such a pair of launches, and the lane-side records they load.
struct PairGrid {
    int64_t workgroups = 0, loads = 0;
};
PairGrid pair_grid(const PairPanel &f, const PairPanel &l);
// Positions of a dof list along a Morton curve of the dofs' places (mesh_expand.cpp).
void morton_order(const bem_mesh &m, int space, const int32_t *dofs, int64_t n, std::vector<int32_t> &order);

// ---------------------------------------------------------------------------
// Errors
void set_error(const std::string &msg);
int fail(int code, const std::string &msg);
#define BEM_HIP_TRY(expr)                                                                   \
    do {                                                                                    \
        hipError_t e_ = (expr);                                                             \
        if (e_ != hipSuccess)                                                               \
            return ::bem::fail(BEM_E_DEVICE, std::string(#expr ": ") + hipGetErrorString(e_)); \
    } while (0)

double now_seconds();

// Gives back the idle part of what is kept between calls: staging slots, pair
// workspaces, dense work areas (capi.cpp).
void release_kept();
// Device and pinned memory; where there is none left, what is kept between calls
// is given back and the allocation tried once more.
hipError_t alloc_device(void **p, size_t bytes);
hipError_t alloc_pinned(void **p, size_t bytes, unsigned flags);

}  // namespace bem

// ---------------------------------------------------------------------------
// Mesh handle (host copies for request expansion and trees, device geometry).
struct bem_mesh {
    int64_t nv = 0, nt = 0;
    int q = 6;
    std::vector<double> xyz;          // nv x 3
    std::vector<int32_t> tri;         // nt x 3
    std::vector<int64_t> star_ptr;    // nv + 1
    std::vector<int32_t> star;        // packed (triangle << 2 | local vertex), ascending triangles
    std::vector<int32_t> dp1_star;    // 3 nt: star-table position of (triangle t, local vertex a) at 3 t + a
    double mean_J = 0.0, mean_edge = 0.0, max_edge = 0.0;
    double box_lo[3] = {0.0, 0.0, 0.0}, box_inv[3] = {0.0, 0.0, 0.0};   // bounding box: low corner, 1/extent
    int max_star = 0;
    int device = 0;
    float *d_g32 = nullptr;
    double *d_g64 = nullptr;
    int4 *d_vtx = nullptr;
    double *d_xyz = nullptr;     // vertices (the singular pairs read them); the allocation holds the next two as well
    int32_t *d_sptr = nullptr;   // star ranges per vertex
    int32_t *d_star = nullptr;   // star table on the device (packed triangle << 2 | local vertex)
    float *d_sgeo = nullptr;     // FP32 record per star entry
    int4 *d_smeta = nullptr;     // vertex ids per star entry, w = local vertex
    size_t dev_bytes = 0;
    std::atomic<int64_t> inflight{0};

    bool adjacent(int64_t a, int64_t b) const {
        const int32_t *ta = &tri[3 * a], *tb = &tri[3 * b];
        for (int i = 0; i < 3; ++i)
            for (int j = 0; j < 3; ++j)
                if (ta[i] == tb[j]) return true;
        return false;
    }
};

namespace bem {

// ---------------------------------------------------------------------------
// Lane side of a request: the triangles the lanes run over, in chunks of at
// most kBlockLanes, and, for P1, the map from each requested lane-side dof to
// its (triangle, local vertex) partial sums.  A P1 chunk holds a run of
// consecutive lane-side dofs together with every triangle of their stars, so
// one workgroup finishes those entries on its own (triangles on a chunk
// border appear in both chunks).  Computed once per dof list; device-resident
// copies are shared by every request of an H-matrix block.
struct LaneSet {
    int64_t ndof = 0;                 // lane-side output positions
    int64_t ndistinct = 0;            // distinct lane triangles (P0: ndof; row form: each once per dof)
    std::vector<int32_t> lane;        // P0: the dofs themselves; P1: triangles, chunk by chunk
    std::vector<int32_t> chunk;       // 4 per chunk: first lane, lanes, first dof, dofs
    std::vector<int32_t> seg_ptr;     // P1: ndof + 1
    std::vector<int32_t> seg;         // P1: packed (slot within the chunk << 2 | local vertex)
    std::vector<int32_t> pos;         // P1: output position of each lane-side dof when the set was
                                      // reordered for locality (empty: identity)
    int64_t nchunk() const { return (int64_t)chunk.size() / 4; }
    // what is staged for the device (block records carry the chunks)
    size_t ints() const { return lane.size() + seg_ptr.size() + seg.size() + pos.size(); }
};

struct LaneRef {                      // device pointers of a resident LaneSet
    const int32_t *lane = nullptr, *seg_ptr = nullptr, *seg = nullptr;
    const int32_t *chunk_host = nullptr;   // the chunk table (host; block records carry it)
    const float *geo = nullptr;            // FP32 records gathered per lane position
    const int4 *meta = nullptr;            // their vertex ids
    int64_t ndof = 0, nlane = 0, nseg = 0, nchunk = 0, ndistinct = 0;
};

// Lane set of a dof list.  With reorder, a P1 list longer than one chunk is
// first ordered along a Morton curve of the vertex positions (ls.pos keeps
// each entry's position in the caller's list): chunks then hold the stars of
// neighbouring vertices instead of whatever the caller's order groups, which
// keeps the duplicated border lanes few.
void build_lane_set(const bem_mesh &m, int space, const int32_t *dofs, int64_t n, LaneSet &ls,
                    bool reorder = false);

// ---------------------------------------------------------------------------
// A request on its way through the server.
struct Request {
    bem_mesh *mesh = nullptr;
    int op = 0, space = 0, prec = 0, near = 0;
    double k = 0.0;
    int64_t nrows = 0, ncols = 0;
    std::vector<int32_t> rows, cols;
    void *out_host = nullptr;   // destination (host); null with borrow = true
    bool borrow = false;        // completion hands out a pointer into pinned staging instead
    const void *result = nullptr;
    void *batch = nullptr;      // batch holding a borrowed result

    // expansion
    int fixrows = 1;            // the fixed items are the request's rows (else its columns)
    int rowfix = 1;             // kernel side: the fixed items are test functions (differs from fixrows
                                // for the adjoint double layer, evaluated as the double layer transposed)
    std::vector<int32_t> fix;   // fixed side: P0 triangles; P1 star ranges [s0, s1) per fixed dof (2 each)
    LaneSet own;                       // lane side, when not external
    const LaneRef *ext = nullptr;      // device-resident lane side
    // the supports of the fixed and lane sides have a positive distance (the
    // blocks of an admissible partition): no pair can share a vertex, so the
    // kernels neither load vertex ids for the lanes nor test for sharing
    bool separated = false;
    int64_t nfix = 0, nlane = 0, nchunk = 0, ndistinct = 0;
    int64_t nstar = 0;          // P1: triangles over the fixed dofs' stars
    size_t elem_bytes = 0;
    size_t in_bytes = 0, out_bytes = 0;
    int64_t evals = 0;          // Q^2 x distinct (fixed, lane) triangle pairs, vertex-sharing pairs included
    int64_t nblocks = 0;
    size_t batch_bytes = 0;     // request_bytes(), cached at expansion

    // staging records built by the submitting thread (prebuild_staging); the
    // server's dispatcher copies them into a batch and fills in what depends
    // on the batch: the request index of each block, the staged inputs, the
    // output and status addresses
    std::vector<NearPair> near_pairs;     // BEM_NEAR_SINGULAR: the request's vertex-sharing pairs
    std::vector<int32_t> near_ints;       // P1: gptr | rptr | rs of NearReq (pair indices within the request);
                                          // the column dofs follow when staged
    int32_t near_slots = 0;               // row-side triangles
    std::vector<int32_t> near_rows;       // P1: rows with at least one pair
    // taken by single triangles or stars whatever its size: one of many in flight that
    // several threads expand, or one whose other form a workspace does not hold
    bool plain = false;
    bool row = false;                     // P1 of few fixed dofs: the row form (build_row_set)
    int32_t tile = 1;                     // P0: fixed triangles per workgroup
    int32_t row_split = 0;                // its log2 shares of a fixed star
    // by triangle pairs (dense.cpp): no lane set and no block table then
    bool paired = false;
    bool pair_error = false;              // under BEM_NEAR_ERROR: two of its triangles share a vertex
    PairPlan pairs;
    int key = 0;                          // launch group (operator, space, precision, rule)
    std::vector<EntryBlock> pre_blocks;   // `req` holds the fixed-side bit only
    ReqDev pre_dev{};

    // completion
    std::mutex mu;
    std::condition_variable cv;
    bool done = false;
    int status = 0;
    double t_submit = 0.0, t_done = 0.0;
    // Completion callback, called from the server's completion thread with all
    // finished requests of one batch that share (on_done, cb_ctx); requests
    // with a callback are not signalled through cv.
    void (*on_done)(Request **, size_t, void *) = nullptr;
    void *cb_ctx = nullptr;
    int64_t tag = 0;            // caller's bookkeeping

    // placement inside a batch
    size_t off_out = 0, off_status = 0;
    bool fast = false;          // written into its batch by the submitter (server fast path)

    int64_t entries() const { return nrows * ncols; }
};

bool is_complex_op(int op);
// Dofs of a space on a mesh: triangles (P0), vertices (P1), 3 x triangles (DP1).
int64_t space_ndof(const bem_mesh &m, int space);
// The entry kernels' space: P0 kernels for P0, the P1 kernels (fixed star
// against lane triangles, per-dof reduction) for P1 and DP1 (a DP1 dof is a
// one-triangle star).
inline int kernel_space(int space) { return space == BEM_P0 ? BEM_P0 : BEM_P1; }
bool is_adjoint_op(int op);
// The operator the entry kernels evaluate: the adjoint double layer runs as
// the double layer with test and trial exchanged.
int kernel_op(int op);
size_t out_elem_bytes(int op, int prec);

// Validate and expand a request (host; runs on the submitting thread).
int expand_request(Request &r, const PairRoom &room = {});
// What a request takes beside its singular pairs as single triangles or stars,
// in bytes (at most, where that is within the limit).
size_t plain_workspace(const Request &r, size_t limit);
// Row form: whether a triangle of a fixed star and one of a lane star share a vertex.
bool row_touches(const Request &r);
// Fast path for requests whose lane side is a resident LaneRef and whose
// fixed side is a single dof known to be valid (H-matrix blocks).
void expand_single_fixed(Request &r, int32_t dof, int rowfix, const LaneRef *ext);

// Device bytes a request needs inside a batch (inputs, outputs, block table).
size_t request_bytes(const Request &r);

// Writes the request's inputs at host_base + off (staging) and fills its
// descriptor with device addresses at dev_base + off; returns the bytes used.
size_t stage_request_inputs(Request &r, char *host_base, char *dev_base, size_t off, ReqDev &d);
// The descriptor fields that do not depend on where the request is staged.
void describe_request(const Request &r, ReqDev &d);
// Copies a request's own lane-side arrays into staging at `off` and points d
// at their device copies (no-op for a device-resident lane side); returns
// the bytes used (r.in_bytes).
size_t stage_own_inputs(const Request &r, char *host_base, char *dev_base, size_t off, ReqDev &d);
// Launch group of a request: (row form or tiles, kernel operator, kernel space, precision, rule).
int request_key(const Request &r);
constexpr int kKeys = 128;
inline Variant key_variant(int key)
{
    return Variant{(key >> 3) & 7, (key >> 2) & 1, (key >> 1) & 1, (key & 1) ? 6 : 4, key >> 6};
}
// Fills r.key, r.pre_blocks and r.pre_dev (called by the submitting thread).
void prebuild_staging(Request &r);
// off_status addresses the request's int32 status word (zeroed by the caller).
void finish_descriptor(const Request &r, char *dev_base, size_t off_out, size_t off_status, ReqDev &d);

// Server
int server_submit(Request *r);
// Room of a request by triangle pairs in the server's slots, beside its entries.
PairRoom server_pair_room(size_t out_bytes);
int server_submit_many(Request *const *rs, size_t n);
// With BEM_DEBUG_TIMING set: prints and resets per-phase host times of the
// dispatch and completion threads (stderr).
void server_print_phases();
int server_wait(Request *r, double timeout_s);
// Status of a finished request handed to a completion callback (requests
// submitted through the server's fast path carry it in the batch).
int server_request_status(const Request *r);
// Completion time of such a request (library clock).
double server_request_done_time(const Request *r);
void server_release(Request *r);           // return a borrowed result
void server_release_batch(void *batch, int n);   // return n borrowed results of one batch (Request::batch)
int server_ensure_started();
bool server_running();

}  // namespace bem
