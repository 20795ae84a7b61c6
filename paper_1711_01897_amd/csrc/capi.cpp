// extern "C" entry points of libbem (declared in include/bem.h).
#include <algorithm>
#include <atomic>
#include <cmath>
#include <new>

#include "bem_internal.hpp"
#include "tree.hpp"

namespace bem {
const char *last_error();
int mesh_create_impl(const double *, int64_t, const int32_t *, int64_t, int, bem_mesh **);
int mesh_destroy_impl(bem_mesh *);
int server_configure(size_t, int);
int server_stats(bem_server_stats_t *, int);
int server_kernel_stats(bem_kernel_stats_t *, int, int *, int);
int aca_block(bem_mesh *, int, int, double, const int32_t *, int64_t, const int32_t *, int64_t, const bem_aca_params *,
              int, void *, void *, int32_t *, int64_t *);
int aca_callback(int64_t, int64_t, int, bem_row_fn, bem_col_fn, void *, const bem_aca_params *, void *, void *,
                 int32_t *);
int hmat_assemble(bem_mesh *, int, int, double, const bem_hmat_params *, bem_hmat **);
int hmat_matvec(const bem_hmat *, const void *, void *);
int hmat_block_info(const bem_hmat *, int64_t, int32_t *, int64_t *, int64_t *, int32_t *, const int32_t **,
                    const int32_t **);
int hmat_block_dense(const bem_hmat *, int64_t, void *);
int hmat_stats(const bem_hmat *, bem_hmat_stats *);
int hmat_destroy(bem_hmat *);
int plan_create(bem_mesh *, int, int, double, const bem_hmat_params *, bem_aca_plan **);
int plan_info(const bem_aca_plan *, int64_t *, int64_t *, double *);
int plan_block(const bem_aca_plan *, int64_t, int64_t *, int64_t *, const int32_t **, const int32_t **);
int plan_run(bem_aca_plan *, const int64_t *, const double *, int64_t, int, bem_aca_run_stats *);
int plans_run(bem_aca_plan *const *, int64_t, const int64_t *, const int64_t *, const double *, int64_t, int, int,
              int, bem_aca_run_stats *);
int plan_factors(const bem_aca_plan *, int64_t, int32_t *, void *, void *);
int plan_destroy(bem_aca_plan *);
void release_dense_kits();
int eval_dense(bem_mesh *, int, int, double, const int32_t *, int64_t, const int32_t *, int64_t, int, int, void *,
               bem_dense_stats *);
}  // namespace bem

using namespace bem;

struct bem_ticket {
    Request req;
};

namespace {

int fill_request(Request &r, bem_mesh *mesh, bem_op op, bem_space space, double k, const int32_t *rows, int64_t nrows,
                 const int32_t *cols, int64_t ncols, bem_prec prec, bem_near near, const PairRoom &room)
{
    if (!mesh) return fail(BEM_E_ARG, "null mesh");
    if (nrows < 0 || ncols < 0) return fail(BEM_E_ARG, "negative request size");
    if ((nrows > 0 && !rows) || (ncols > 0 && !cols)) return fail(BEM_E_ARG, "null index array");
    r.mesh = mesh;
    r.op = op;
    r.space = space;
    r.prec = prec;
    r.near = near;
    r.k = k;
    r.nrows = nrows;
    r.ncols = ncols;
    r.rows.assign(rows, rows + nrows);
    r.cols.assign(cols, cols + ncols);
    return expand_request(r, room);
}

// Room for the pairs of a served request; sizes that fill_request refuses, and
// entries past any slot, have none.
PairRoom served_room(int op, int prec, int64_t nrows, int64_t ncols)
{
    if (nrows <= 0 || ncols <= 0 || nrows > INT32_MAX || ncols > INT32_MAX) return {};
    const size_t n = (size_t)nrows * (size_t)ncols;
    return n > SIZE_MAX / 16 ? PairRoom{} : server_pair_room(n * out_elem_bytes(op, prec));
}

// Staging of the async path: a pinned host image of the request and device
// workspace of the same size, kept from call to call.  A slot carries the
// event recorded after the last kernel that reads it and is taken again, by
// any thread and stream, only once the host has seen that event complete, so
// no call waits for one: with every slot in flight, on a capturing stream or for a
// request larger than a slot the call allocates its own (below).  Allocating
// per call was what a small request cost: one row of 97 entries took 96
// us, 19 us with a kept slot.
// Slots are released when the last mesh is destroyed.
constexpr size_t kSlotLeast = size_t(64) << 10, kSlotMost = size_t(8) << 20;   // bytes, powers of two between
constexpr size_t kSlotsTotal = size_t(128) << 20;                            // pinned bytes over all slots
constexpr size_t kSlotsMost = 64;
constexpr size_t kPairBudget = size_t(256) << 20;   // workspace of one request by triangle pairs (larger ones go in panels)
constexpr size_t kWorkTotal = size_t(1) << 30;      // of all that are kept
// The same for the no-allocation entry point, behind the rest of its workspace.  16
// MiB within the 32 of the rest cut blocks into so many panels that they took two
// to three times what their stars do (pairs_pay has the figures).
constexpr size_t kNoAllocBytes = size_t(32) << 20, kNoAllocPairs = size_t(64) << 20;

struct StageSlot {
    char *host = nullptr;       // pinned
    char *host_dev = nullptr;   // its device address
    char *dev = nullptr;
    size_t bytes = 0;
    int device = 0;
    hipEvent_t done = nullptr;
    bool taken = false;
    bool recorded = false;      // `done` has been recorded since the slot was made
};

std::mutex g_stage_mu;
std::vector<StageSlot *> g_slots;
size_t g_slots_bytes = 0;

// Workspaces of requests by triangle pairs (local matrices).  Calls on one
// stream follow each other there, so they share one: a call takes the buffer
// last used on its stream behind that use (the stream waits for its event,
// which on the same stream costs nothing), else one whose last use the host has
// seen end, else a new one within the total.
struct WorkBuf {
    char *p = nullptr;
    size_t bytes = 0;
    int device = 0;
    hipStream_t last = nullptr;
    hipEvent_t done = nullptr;
    bool taken = false, recorded = false;
};
std::vector<WorkBuf *> g_works;
size_t g_works_bytes = 0;

bool finished(hipEvent_t e)
{
    if (hipEventQuery(e) == hipSuccess) return true;
    (void)hipGetLastError();   // "not ready" is no error of the launch that follows
    return false;
}

void destroy_slot(StageSlot *x)
{
    if (x->done) (void)hipEventDestroy(x->done);
    if (x->host) (void)hipHostFree(x->host);
    if (x->dev) (void)hipFree(x->dev);
    delete x;
}

void destroy_work(WorkBuf *w)
{
    if (w->done) (void)hipEventDestroy(w->done);
    if (w->p) (void)hipFree(w->p);
    delete w;
}

// A workspace of at least `bytes` for work about to be enqueued on s, or null.
WorkBuf *take_work(size_t bytes, int device, hipStream_t s)
{
    std::lock_guard<std::mutex> g(g_stage_mu);
    WorkBuf *idle = nullptr;
    for (WorkBuf *w : g_works) {
        if (w->taken || w->device != device || w->bytes < bytes) continue;
        if (w->recorded && w->last == s) {
            if (hipStreamWaitEvent(s, w->done, 0) != hipSuccess) {
                (void)hipGetLastError();
                continue;
            }
            w->taken = true;
            return w;
        }
        if (!idle && (!w->recorded || finished(w->done))) idle = w;
    }
    if (idle) {
        idle->taken = true;
        return idle;
    }
    size_t cap = size_t(1) << 20;
    while (cap < bytes) cap *= 2;
    // smaller ones that nothing uses make room
    for (size_t i = 0; i < g_works.size() && g_works_bytes + cap > kWorkTotal;) {
        WorkBuf *w = g_works[i];
        if (w->taken || (w->recorded && !finished(w->done))) {
            ++i;
            continue;
        }
        g_works_bytes -= w->bytes;
        destroy_work(w);
        g_works[i] = g_works.back();
        g_works.pop_back();
    }
    if (g_works_bytes + cap > kWorkTotal) return nullptr;
    WorkBuf *w = new (std::nothrow) WorkBuf();
    if (!w) return nullptr;
    if (hipMalloc((void **)&w->p, cap) != hipSuccess ||
        hipEventCreateWithFlags(&w->done, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        destroy_work(w);
        return nullptr;
    }
    w->bytes = cap;
    w->device = device;
    w->taken = true;
    g_works.push_back(w);
    g_works_bytes += cap;
    return w;
}

// Returns a workspace whose last use has been enqueued on s (or not at all).
hipError_t give_work(WorkBuf *w, hipStream_t s, bool enqueued)
{
    hipError_t e = hipSuccess;
    if (enqueued) {
        e = hipEventRecord(w->done, s);
        if (e != hipSuccess) (void)hipStreamSynchronize(s);
    }
    std::lock_guard<std::mutex> g(g_stage_mu);
    if (enqueued && e == hipSuccess) {
        w->recorded = true;
        w->last = s;
    }
    w->taken = false;
    return e;
}

// A slot of at least `bytes` on `device` that no enqueued work uses, or null.
StageSlot *take_slot(size_t bytes, int device)
{
    if (bytes > kSlotMost) return nullptr;
    size_t cap = kSlotLeast;
    while (cap < bytes) cap *= 2;
    std::lock_guard<std::mutex> g(g_stage_mu);
    StageSlot *x = nullptr;   // the smallest that holds them
    for (StageSlot *y : g_slots)
        if (!y->taken && y->device == device && y->bytes >= bytes && (!x || y->bytes < x->bytes) &&
            (!y->recorded || finished(y->done)))
            x = y;
    if (x) {
        x->taken = true;
        return x;
    }
    // At a limit idle smaller slots make room.  That waits for the device once,
    // where allocating its own would cost this request and every later one: after a
    // burst of 64 small requests one of 200 KB took 93 us a call instead of 29.
    auto full = [&] { return g_slots.size() >= kSlotsMost || g_slots_bytes + cap > kSlotsTotal; };
    for (size_t i = 0; i < g_slots.size() && full();) {
        StageSlot *y = g_slots[i];
        if (y->taken || y->bytes >= cap || (y->recorded && !finished(y->done))) {
            ++i;
            continue;
        }
        g_slots_bytes -= y->bytes;
        destroy_slot(y);
        g_slots[i] = g_slots.back();
        g_slots.pop_back();
    }
    if (full()) return nullptr;
    x = new (std::nothrow) StageSlot();
    if (!x) return nullptr;
    x->bytes = cap;
    x->device = device;
    if (hipHostMalloc((void **)&x->host, cap, hipHostMallocDefault) != hipSuccess ||
        hipHostGetDevicePointer((void **)&x->host_dev, x->host, 0) != hipSuccess ||
        hipMalloc((void **)&x->dev, cap) != hipSuccess ||
        hipEventCreateWithFlags(&x->done, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        destroy_slot(x);
        return nullptr;
    }
    x->taken = true;
    g_slots.push_back(x);
    g_slots_bytes += cap;
    return x;
}

// Returns a slot whose last use has been enqueued on s (enqueued = false:
// nothing was).
hipError_t give_slot(StageSlot *x, hipStream_t s, bool enqueued)
{
    hipError_t e = hipSuccess;
    if (enqueued) {
        e = hipEventRecord(x->done, s);
        // without the event the work is waited for: the slot must not be reused before
        if (e != hipSuccess) (void)hipStreamSynchronize(s);
    }
    std::lock_guard<std::mutex> g(g_stage_mu);
    if (enqueued && e == hipSuccess) x->recorded = true;
    x->taken = false;
    return e;
}

// Pinned staging of the calls that allocate their own.  A buffer is freed
// once the event recorded after its copy has completed; completed buffers are
// reclaimed on later such calls (or immediately when no event could be
// recorded).
std::vector<std::pair<hipEvent_t, char *>> g_stage_pending;

void reclaim_stages()
{
    std::lock_guard<std::mutex> g(g_stage_mu);
    auto it = g_stage_pending.begin();
    while (it != g_stage_pending.end()) {
        if (finished(it->first)) {
            (void)hipEventDestroy(it->first);
            (void)hipHostFree(it->second);
            it = g_stage_pending.erase(it);
        } else {
            ++it;
        }
    }
}

char *pinned_stage(size_t bytes)
{
    reclaim_stages();
    char *p = nullptr;
    if (alloc_pinned((void **)&p, bytes, hipHostMallocDefault) != hipSuccess) return nullptr;
    return p;
}

void pinned_release(char *p, hipEvent_t after)
{
    if (!after) {
        // nothing was enqueued that reads p
        (void)hipHostFree(p);
        return;
    }
    std::lock_guard<std::mutex> g(g_stage_mu);
    g_stage_pending.push_back({after, p});
}

// Meshes alive; the last one's end releases the slots that are not in use.
std::atomic<int64_t> g_meshes{0};

void release_slots()
{
    std::lock_guard<std::mutex> g(g_stage_mu);
    for (size_t i = 0; i < g_slots.size();) {
        StageSlot *x = g_slots[i];
        if (x->taken || (x->recorded && !finished(x->done))) {
            ++i;
            continue;
        }
        g_slots_bytes -= x->bytes;
        destroy_slot(x);
        g_slots[i] = g_slots.back();
        g_slots.pop_back();
    }
    for (size_t i = 0; i < g_works.size();) {
        WorkBuf *w = g_works[i];
        if (w->taken || (w->recorded && !finished(w->done))) {
            ++i;
            continue;
        }
        g_works_bytes -= w->bytes;
        destroy_work(w);
        g_works[i] = g_works.back();
        g_works.pop_back();
    }
}

// Requests of at most this many workgroups read their descriptor, block
// records and lists straight from the pinned image: a workgroup waits for a
// few host-link reads, less than a copy kernel and the gap behind it take.
// Back to back a call takes 12.0-12.7 us that way and 14.7-15.7 with the copy (P0 1 x
// 256 to 8 x 1,024, P1 1 x 8 to 8 x 32), one that is waited for 1 us more (25 for
// 24).  There is no edge: up to 256 workgroups it is the same; but with more of them the
// same lists cross the link once per fixed item, so the line stays at rows and columns.
constexpr int64_t kDirectBlocks = 32;

// A block by triangle pairs whose workspace the device does not have.
constexpr int kNoRoom = 1;

// Enqueues an expanded request on `s` with its result in device memory
// dev_out (kNoRoom: nothing enqueued, to be asked for by stars).  Workspace layout: descriptor | block table | singular pairs |
// inputs | status word, staged in one host image.  With fixed == nullptr image
// and workspace are a kept slot's, the image copied to the workspace by a
// kernel or, for a few workgroups, read in place; or both are allocated for the
// call (stream-ordered workspace, pinned image released once its copy has
// completed).  Otherwise both live in fixed memory: the workspace is `fixed`
// (fixed_bytes long and kNoAllocPairs for local matrices; larger requests fail), the host image a per-thread
// pageable buffer whose copy completes before the call returns (a pageable
// host-to-device copy is synchronous with the host).
int enqueue_device_request(Request &r, void *dev_out, hipStream_t s, char *fixed, size_t fixed_bytes)
{
    bem_mesh *mesh = r.mesh;
    if (r.near == BEM_NEAR_ERROR) {
        // host-side check: nothing may be enqueued for a failing request
        if (r.paired) {
            if (r.pair_error) return fail(BEM_E_NEARFIELD, "a contributing triangle pair shares a vertex");
        } else if (r.row) {
            if (row_touches(r)) return fail(BEM_E_NEARFIELD, "a contributing triangle pair shares a vertex");
        } else if (r.space == BEM_P0) {
            for (int32_t a : r.rows)
                for (int32_t b : r.cols)
                    if (mesh->adjacent(a, b)) return fail(BEM_E_NEARFIELD, "a contributing triangle pair shares a vertex");
        } else {
            for (size_t f = 0; 2 * f + 1 < r.fix.size(); ++f)
                for (int32_t st = r.fix[2 * f]; st < r.fix[2 * f + 1]; ++st)
                    for (int32_t t : r.own.lane)
                        if (mesh->adjacent(mesh->star[st] >> 2, t))
                            return fail(BEM_E_NEARFIELD, "a contributing triangle pair shares a vertex");
        }
    }
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    size_t off = 0;
    const size_t off_req = off;
    off = al(off + sizeof(ReqDev));
    const size_t off_b = off;
    off = al(off + sizeof(EntryBlock) * (size_t)r.nblocks);
    const size_t off_near = off;
    const bool near = !r.near_pairs.empty();
    const NearCount near_n = near_count(r);
    const NearLayout near_l = near_layout(near_kind(r), near_n);
    off = al(off + (near ? near_l.staged : 0));
    const size_t off_in = off;
    off = al(off + (r.paired ? 4 * r.pairs.ints.size() : r.in_bytes));
    const size_t off_status = off;
    off = al(off + 8);
    const size_t in_total = off;
    // what the singular kernels write for each other follows the staged part
    const size_t ws_staged = in_total + (near ? near_l.bytes - near_l.staged : 0);
    // the local matrices of a request by triangle pairs: with a slot a kept
    // workspace of their own, in the fixed memory at its end, else behind the rest
    const size_t work_bytes = r.paired ? r.pairs.work : 0;
    const size_t work_at = fixed ? fixed_bytes : al(ws_staged), ws_total = al(ws_staged) + work_bytes;
    // the limit is that of the plain forms, whichever form the request takes
    const size_t needed = fixed ? std::max(ws_staged, plain_workspace(r, fixed_bytes)) : 0;
    if (needed > fixed_bytes || (fixed && work_bytes > kNoAllocPairs))
        return fail(BEM_E_OOM, "request needs " + std::to_string(needed) + " bytes of workspace, more than the " +
                                   std::to_string(fixed_bytes) + "-byte static workspace of the no-allocation entry point");
    char *host = nullptr;
    char *ws = fixed;
    StageSlot *slot = nullptr;
    WorkBuf *wbuf = nullptr;
    thread_local std::vector<char> pageable;
    if (fixed) {
        pageable.assign(in_total, 0);
        host = pageable.data();
    } else {
        int cur = -1, dev = -1;
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipGetDevice(&cur) == hipSuccess && hipStreamGetDevice(s, &dev) == hipSuccess && cur == dev &&
            hipStreamIsCapturing(s, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone)
            slot = take_slot(ws_staged, dev);
        else
            (void)hipGetLastError();
        if (slot && work_bytes && !(wbuf = take_work(work_bytes, dev, s))) {
            (void)give_slot(slot, s, false);
            slot = nullptr;
        }
        if (slot) {
            host = slot->host;
            ws = slot->dev;
        } else {
            host = pinned_stage(in_total);
            if (!host) return fail(BEM_E_OOM, "pinned staging allocation failed");
            std::memset(host, 0, in_total);
            hipError_t e = hipMallocAsync((void **)&ws, ws_total, s);
            if (e == hipErrorOutOfMemory) {
                (void)hipGetLastError();
                release_kept();
                e = hipMallocAsync((void **)&ws, ws_total, s);
            }
            if (e != hipSuccess) {
                (void)hipGetLastError();   // reported here, not by the next launch
                pinned_release(host, nullptr);
                if (e == hipErrorOutOfMemory && r.paired) return kNoRoom;
                return fail(BEM_E_DEVICE, std::string("hipMallocAsync: ") + hipGetErrorString(e));
            }
        }
    }
    // where the kernels read the staged image
    const bool direct = slot && !near && !r.paired && r.nblocks <= kDirectBlocks;
    char *work = wbuf ? wbuf->p : ws + work_at;
    char *img = direct ? slot->host_dev : ws;
    if (r.paired) {
        std::memcpy(host + off_in, r.pairs.ints.data(), 4 * r.pairs.ints.size());
    } else {
        ReqDev d;
        stage_request_inputs(r, host, img, off_in, d);
        finish_descriptor(r, img, 0, off_status, d);
        d.out = dev_out;
        std::memcpy(host + off_req, &d, sizeof(ReqDev));
        write_blocks(r, 0, reinterpret_cast<EntryBlock *>(host + off_b));
    }
    NearLayout nl = near_l;
    if (near) {
        // the device-only part sits past the staged image of the whole request
        nl.keys += in_total - off_near - near_l.staged;
        nl.local += in_total - off_near - near_l.staged;
        NearCount at;
        stage_near(r, nl, host + off_near, ws + off_near, static_cast<char *>(dev_out), at);
    }
    *reinterpret_cast<int64_t *>(host + off_status) = 0;
    hipError_t e = hipSuccess;
    if (slot) {
        if (!direct) e = launch_stage_copy(slot->host_dev, ws, in_total, s);
        if (e != hipSuccess) {
            (void)give_slot(slot, s, false);
            if (wbuf) (void)give_work(wbuf, s, false);
        }
    } else {
        e = hipMemcpyAsync(ws, host, in_total, hipMemcpyHostToDevice, s);
        if (!fixed) {
            hipEvent_t ev = nullptr;
            if (e == hipSuccess) e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
            if (e == hipSuccess) e = hipEventRecord(ev, s);
            pinned_release(host, e == hipSuccess ? ev : nullptr);
        }
    }
    if (e != hipSuccess) return fail(BEM_E_DEVICE, std::string("staging copy: ") + hipGetErrorString(e));
    const ReqDev *dreq = (const ReqDev *)(img + off_req);
    const Variant v{kernel_op(r.op), r.space, r.prec, mesh->q, r.row || r.tile > 1 ? 1 : 0};
    if (r.paired) {
        const int64_t sf = r.fixrows ? r.ncols : 1, sl = r.fixrows ? 1 : r.ncols;
        for (const PairPanel &f : r.pairs.fix)
            for (const PairPanel &l : r.pairs.lane)
                if (e == hipSuccess)
                    e = launch_pairs(*mesh, r.pairs, f, l, (const int32_t *)(ws + off_in), work, dev_out, sf, sl, r.k, s);
    } else {
        e = launch_entries(v, dreq, (const EntryBlock *)(img + off_b), r.nblocks, s);
    }
    if (e == hipSuccess && near) e = launch_near(near_kind(r), nl, near_n, ws + off_near, s);
    if (slot) {
        hipError_t g = wbuf ? give_work(wbuf, s, true) : hipSuccess;
        if (e == hipSuccess) e = g;
        g = give_slot(slot, s, true);
        if (e == hipSuccess) e = g;
    } else if (!fixed && e == hipSuccess) {
        e = hipFreeAsync(ws, s);
    }
    if (e != hipSuccess) return fail(BEM_E_DEVICE, std::string("request launch: ") + hipGetErrorString(e));
    return BEM_OK;
}

// Workspace of bem_eval_entries_async_noalloc: one request's descriptor,
// block table, singular-pair records, inputs and status word, and behind them the
// local matrices of a block by triangle pairs.  Each device
// the library runs on holds its own copy for the life of the process; host
// code reaches it only through the address hipGetSymbolAddress returns for
// that device.
__device__ __align__(256) char scratch[kNoAllocBytes + kNoAllocPairs];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char *g_scratch_ptr[kMaxDevices] = {};

// The device address of `scratch` on `device`, looked up once per device
// with that device current (the previous current device is restored).
int noalloc_workspace(int device, char **out)
{
    if (device < 0 || device >= kMaxDevices) return fail(BEM_E_ARG, "device ordinal out of range");
    std::lock_guard<std::mutex> g(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        int cur = 0;
        BEM_HIP_TRY(hipGetDevice(&cur));
        if (cur != device) BEM_HIP_TRY(hipSetDevice(device));
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (cur != device) (void)hipSetDevice(cur);
        if (e != hipSuccess || !p)
            return fail(BEM_E_DEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        g_scratch_ptr[device] = static_cast<char *>(p);
    }
    *out = g_scratch_ptr[device];
    return BEM_OK;
}

}  // namespace

namespace bem {

void release_kept()
{
    release_slots();
    release_dense_kits();
}

hipError_t alloc_device(void **p, size_t bytes)
{
    hipError_t e = hipMalloc(p, bytes);
    if (e != hipErrorOutOfMemory) return e;
    (void)hipGetLastError();   // no error of a later launch
    release_kept();
    e = hipMalloc(p, bytes);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

hipError_t alloc_pinned(void **p, size_t bytes, unsigned flags)
{
    hipError_t e = hipHostMalloc(p, bytes, flags);
    if (e != hipErrorOutOfMemory) return e;
    (void)hipGetLastError();
    release_kept();
    e = hipHostMalloc(p, bytes, flags);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

}  // namespace bem

extern "C" {

const char *bem_last_error(void) { return bem::last_error(); }

int bem_mesh_create(const double *xyz, int64_t nv, const int32_t *tri, int64_t nt, int quad_points, bem_mesh **out)
{
    const int rc = mesh_create_impl(xyz, nv, tri, nt, quad_points, out);
    if (rc == BEM_OK) g_meshes.fetch_add(1);
    return rc;
}

int bem_mesh_destroy(bem_mesh *mesh)
{
    const int rc = mesh_destroy_impl(mesh);
    if (rc == BEM_OK && g_meshes.fetch_sub(1) == 1) release_kept();
    return rc;
}

int bem_mesh_info(const bem_mesh *m, bem_mesh_info_t *info)
{
    if (!m || !info) return fail(BEM_E_ARG, "null argument");
    info->nv = m->nv;
    info->nt = m->nt;
    info->quad_points = m->q;
    info->max_star = m->max_star;
    info->mean_jacobian = m->mean_J;
    info->mean_edge = m->mean_edge;
    info->device_bytes = m->dev_bytes;
    return BEM_OK;
}

int bem_eval_entries(bem_mesh *mesh, bem_op op, bem_space space, double k, const int32_t *rows, int64_t nrows,
                     const int32_t *cols, int64_t ncols, bem_prec prec, bem_near near, void *out)
{
    Request *r = new (std::nothrow) Request();
    if (!r) return fail(BEM_E_OOM, "host allocation failed");
    int rc = fill_request(*r, mesh, op, space, k, rows, nrows, cols, ncols, prec, near, served_room(op, prec, nrows, ncols));
    if (rc == BEM_OK && r->entries() > 0) {
        if (!out) {
            rc = fail(BEM_E_ARG, "null output");
        } else {
            r->out_host = out;
            rc = server_submit(r);
            if (rc == BEM_OK) {
                rc = server_wait(r, -1.0);
                if (rc == BEM_E_NEARFIELD) fail(rc, "a contributing triangle pair shares a vertex");
            }
        }
    }
    delete r;
    return rc;
}

int bem_submit(bem_mesh *mesh, bem_op op, bem_space space, double k, const int32_t *rows, int64_t nrows,
               const int32_t *cols, int64_t ncols, bem_prec prec, bem_near near, void *out, bem_ticket **ticket)
{
    if (!ticket) return fail(BEM_E_ARG, "null ticket");
    bem_ticket *t = new (std::nothrow) bem_ticket();
    if (!t) return fail(BEM_E_OOM, "host allocation failed");
    Request &r = t->req;
    int rc = fill_request(r, mesh, op, space, k, rows, nrows, cols, ncols, prec, near, served_room(op, prec, nrows, ncols));
    if (rc == BEM_OK) {
        if (r.entries() == 0) {
            r.done = true;
            r.status = BEM_OK;
            r.t_submit = r.t_done = now_seconds();
        } else if (!out) {
            rc = fail(BEM_E_ARG, "null output");
        } else {
            r.out_host = out;
            rc = server_submit(&r);
        }
    }
    if (rc != BEM_OK) {
        delete t;
        return rc;
    }
    *ticket = t;
    return BEM_OK;
}

int bem_ticket_wait(bem_ticket *t, double timeout_s)
{
    if (!t) return fail(BEM_E_ARG, "null ticket");
    const int rc = server_wait(&t->req, timeout_s);
    if (rc == BEM_E_NEARFIELD) fail(rc, "a contributing triangle pair shares a vertex");
    return rc;
}

int bem_ticket_times(const bem_ticket *t, double *t_submit, double *t_done)
{
    if (!t) return fail(BEM_E_ARG, "null ticket");
    if (t_submit) *t_submit = t->req.t_submit;
    if (t_done) *t_done = t->req.t_done;
    return BEM_OK;
}

int bem_ticket_free(bem_ticket *t)
{
    if (!t) return BEM_OK;
    (void)server_wait(&t->req, -1.0);
    delete t;
    return BEM_OK;
}

int bem_eval_entries_async(bem_mesh *mesh, bem_op op, bem_space space, double k, const int32_t *rows, int64_t nrows,
                           const int32_t *cols, int64_t ncols, bem_prec prec, bem_near near, void *dev_out,
                           void *stream)
{
    Request r;
    int rc = fill_request(r, mesh, op, space, k, rows, nrows, cols, ncols, prec, near, {kPairBudget});
    if (rc != BEM_OK) return rc;
    if (r.entries() == 0) return BEM_OK;
    if (!dev_out) return fail(BEM_E_ARG, "null output");
    rc = enqueue_device_request(r, dev_out, (hipStream_t)stream, nullptr, 0);
    if (rc == kNoRoom) {
        r.plain = true;
        rc = expand_request(r);
        if (rc == BEM_OK) rc = enqueue_device_request(r, dev_out, (hipStream_t)stream, nullptr, 0);
    }
    return rc;
}

int bem_eval_entries_async_noalloc(bem_mesh *mesh, bem_op op, bem_space space, double k, const int32_t *rows,
                                   int64_t nrows, const int32_t *cols, int64_t ncols, bem_prec prec, bem_near near,
                                   void *dev_out, void *stream)
{
    Request r;
    int rc = fill_request(r, mesh, op, space, k, rows, nrows, cols, ncols, prec, near, {kNoAllocPairs});
    if (rc != BEM_OK) return rc;
    if (r.entries() == 0) return BEM_OK;
    if (!dev_out) return fail(BEM_E_ARG, "null output");
    char *ws = nullptr;
    rc = noalloc_workspace(mesh->device, &ws);
    if (rc != BEM_OK) return rc;
    rc = enqueue_device_request(r, dev_out, (hipStream_t)stream, ws, kNoAllocBytes);
    if (rc == BEM_E_OOM && (r.paired || r.row)) {
        // by stars it may still fit
        r.plain = true;
        rc = expand_request(r);
        if (rc == BEM_OK) rc = enqueue_device_request(r, dev_out, (hipStream_t)stream, ws, kNoAllocBytes);
    }
    return rc;
}

int bem_server_config(size_t arena_bytes, int max_batch_requests)
{
    return server_configure(arena_bytes, max_batch_requests);
}

int bem_server_stats(bem_server_stats_t *stats, int reset)
{
    if (!stats) return fail(BEM_E_ARG, "null argument");
    return server_stats(stats, reset);
}

int bem_server_kernel_stats(bem_kernel_stats_t *out, int max_entries, int *count, int reset)
{
    if (max_entries < 0 || !count) return fail(BEM_E_ARG, "bad arguments");
    return server_kernel_stats(out, max_entries, count, reset);
}

int bem_aca_block(bem_mesh *mesh, bem_op op, bem_space space, double k, const int32_t *rows, int64_t m,
                  const int32_t *cols, int64_t n, const bem_aca_params *params, bem_prec prec, void *U, void *V,
                  int32_t *rank, int64_t *entries_evaluated)
{
    return aca_block(mesh, op, space, k, rows, m, cols, n, params, prec, U, V, rank, entries_evaluated);
}

int bem_aca_callback(int64_t m, int64_t n, int is_complex, bem_row_fn get_row, bem_col_fn get_col, void *ctx,
                     const bem_aca_params *params, void *U, void *V, int32_t *rank)
{
    return aca_callback(m, n, is_complex, get_row, get_col, ctx, params, U, V, rank);
}

int bem_partition(const double *xyz, int64_t nv, const int32_t *tri, int64_t nt, bem_space space, int32_t leaf_size,
                  double eta, int32_t max_block, int32_t *perm, int32_t *cl_begin, int32_t *cl_end, int64_t max_clusters, int32_t *blocks,
                  int64_t max_blocks, int64_t *nclusters, int64_t *nblocks)
{
    if (!xyz || !tri || nv < 1 || nt < 1 || leaf_size < 1 || !(eta > 0) || max_block < 0 || !nclusters || !nblocks)
        return fail(BEM_E_ARG, "bad partition arguments");
    if (space != BEM_P0 && space != BEM_P1 && space != BEM_DP1) return fail(BEM_E_ARG, "unknown space");
    for (int64_t i = 0; i < 3 * nt; ++i)
        if (tri[i] < 0 || tri[i] >= nv) return fail(BEM_E_ARG, "triangle vertex index out of range");
    bem_mesh m;
    m.nv = nv;
    m.nt = nt;
    m.xyz.assign(xyz, xyz + 3 * nv);
    m.tri.assign(tri, tri + 3 * nt);
    std::vector<double> pts, slo, shi;
    dof_geometry(m, space, pts, slo, shi);
    Partition P;
    build_partition(pts, slo, shi, leaf_size, eta, max_block, P);
    *nclusters = (int64_t)P.nodes.size();
    *nblocks = (int64_t)P.blocks.size();
    if ((int64_t)P.nodes.size() > max_clusters || (int64_t)P.blocks.size() > max_blocks)
        return fail(BEM_E_ARG, "capacity too small");
    if (perm) std::copy(P.perm.begin(), P.perm.end(), perm);
    for (size_t c = 0; c < P.nodes.size(); ++c) {
        if (cl_begin) cl_begin[c] = (int32_t)P.nodes[c].begin;
        if (cl_end) cl_end[c] = (int32_t)P.nodes[c].end;
    }
    if (blocks)
        for (size_t b = 0; b < P.blocks.size(); ++b) {
            blocks[3 * b] = P.blocks[b].tau;
            blocks[3 * b + 1] = P.blocks[b].sigma;
            blocks[3 * b + 2] = P.blocks[b].admissible;
        }
    return BEM_OK;
}

int bem_hmat_assemble(bem_mesh *mesh, bem_op op, bem_space space, double k, const bem_hmat_params *params,
                      bem_hmat **out)
{
    return hmat_assemble(mesh, op, space, k, params, out);
}

int bem_hmat_matvec(const bem_hmat *h, const void *x, void *y) { return hmat_matvec(h, x, y); }

int bem_hmat_stats_get(const bem_hmat *h, bem_hmat_stats *stats) { return hmat_stats(h, stats); }

int bem_hmat_block_info(const bem_hmat *h, int64_t b, int32_t *admissible, int64_t *m, int64_t *n, int32_t *rank,
                        const int32_t **rows, const int32_t **cols)
{
    return hmat_block_info(h, b, admissible, m, n, rank, rows, cols);
}

int bem_hmat_block_dense(const bem_hmat *h, int64_t b, void *out) { return hmat_block_dense(h, b, out); }

int bem_hmat_destroy(bem_hmat *h) { return hmat_destroy(h); }

int bem_aca_plan_create(bem_mesh *mesh, bem_op op, bem_space space, double k, const bem_hmat_params *params,
                        bem_aca_plan **out)
{
    return plan_create(mesh, op, space, k, params, out);
}

int bem_aca_plan_info(const bem_aca_plan *plan, int64_t *n_blocks, int64_t *ndof, double *setup_seconds)
{
    return plan_info(plan, n_blocks, ndof, setup_seconds);
}

int bem_aca_plan_block(const bem_aca_plan *plan, int64_t b, int64_t *m, int64_t *n, const int32_t **rows,
                       const int32_t **cols)
{
    return plan_block(plan, b, m, n, rows, cols);
}

int bem_aca_plan_run(bem_aca_plan *plan, const int64_t *blocks, const double *arrival, int64_t n, bem_prec prec,
                     bem_aca_run_stats *stats)
{
    return plan_run(plan, blocks, arrival, n, prec, stats);
}

int bem_aca_plans_run(bem_aca_plan *const *plans, int64_t nplans, const int64_t *plan_index, const int64_t *blocks,
                      const double *arrival, int64_t n, bem_prec prec, int32_t n_workers, int32_t blocks_per_worker,
                      bem_aca_run_stats *stats)
{
    return plans_run(plans, nplans, plan_index, blocks, arrival, n, prec, n_workers, blocks_per_worker, stats);
}

int bem_aca_plan_factors(const bem_aca_plan *plan, int64_t b, int32_t *rank, void *U, void *V)
{
    return plan_factors(plan, b, rank, U, V);
}

int bem_aca_plan_destroy(bem_aca_plan *plan) { return plan_destroy(plan); }

int bem_eval_dense(bem_mesh *mesh, bem_op op, bem_space space, double k, const int32_t *rows, int64_t nrows,
                   const int32_t *cols, int64_t ncols, bem_prec prec, bem_near near, void *out, bem_dense_stats *stats)
{
    if (nrows > 0 && ncols > 0 && !out) return fail(BEM_E_ARG, "null output");
    return eval_dense(mesh, op, space, k, rows, nrows, cols, ncols, prec, near, out, stats);
}

}  // extern "C"
