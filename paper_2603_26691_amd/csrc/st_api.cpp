// C ABI of the scaletrack library: argument validation, buffer ownership and
// the order of kernel launches.  Every entry point returns an st_status and
// catches everything; nothing throws or aborts across the boundary.
#include <hip/hip_runtime.h>

#include <math.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "st_internal.h"

// ---------------------------------------------------------------------------
// device memory
// ---------------------------------------------------------------------------
namespace st {
namespace {

// Blocks kept for the next context: at most kKeepBytes in all, for all devices
// and threads, and none that the last kKeepFrees calls of block_free have passed
// by; all of them are given back when one of the library's allocations finds no
// memory, and by st_release_memory.  Making
// and freeing device memory can cost more than a short-lived context's work:
// memory is cleared on its way through the driver, so a program that makes a
// context per iteration waits for that.  3e6 droplets put in, read back and
// closed: 5.1 ms with an allocation per array (4.1 ms of them in hipFree), 22.6
// ms in a process that has just freed large buffers; 1.1 ms with kept blocks.
constexpr size_t kKeepBytes = (size_t)512 << 20;
constexpr uint64_t kKeepFrees = 512;

struct Kept {
    int device;
    Block b;
    uint64_t at;     // the count of block_free calls when it was kept
};
struct Keeper {
    std::mutex mu;
    std::vector<Kept> kept;   // oldest first
    size_t bytes = 0;
    uint64_t frees = 0;
};
// (never destroyed: contexts may be closed while the process ends)
Keeper &keeper()
{
    static Keeper *const k = new Keeper();
    return *k;
}

void drop(Keeper &k, size_t i)
{
    (void)hipFree(k.kept[i].b.buf);
    k.bytes -= k.kept[i].b.bytes;
    k.kept.erase(k.kept.begin() + (ptrdiff_t)i);
}

}  // namespace

void release_kept()
{
    Keeper &k = keeper();
    std::lock_guard<std::mutex> lock(k.mu);
    while (!k.kept.empty()) drop(k, 0);
}

hipError_t device_malloc(void **p, size_t bytes)
{
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        release_kept();
        e = hipMalloc(p, bytes);
    }
    if (e != hipSuccess) (void)hipGetLastError();   // reported here, not by the next launch
    return e;
}

hipError_t block_alloc(int device, size_t bytes, Block *out)
{
    if (bytes == 0) bytes = 8;
    if (bytes <= kKeepBytes) {
        Keeper &k = keeper();
        std::lock_guard<std::mutex> lock(k.mu);
        // the smallest that fits and wastes at most a quarter
        size_t best = k.kept.size();
        for (size_t i = 0; i < k.kept.size(); ++i) {
            const Kept &e = k.kept[i];
            if (e.device == device && e.b.bytes >= bytes && e.b.bytes <= bytes + bytes / 4 &&
                (best == k.kept.size() || e.b.bytes < k.kept[best].b.bytes))
                best = i;
        }
        if (best < k.kept.size()) {
            *out = k.kept[best].b;
            k.bytes -= out->bytes;
            k.kept.erase(k.kept.begin() + (ptrdiff_t)best);
            return hipSuccess;
        }
    }
    void *p = nullptr;
    const hipError_t e = device_malloc(&p, bytes);
    if (e == hipSuccess) *out = Block{p, bytes};
    return e;
}

void block_free(int device, Block *b)
{
    if (!b->buf) return;
    const Block mine = *b;
    *b = Block{};
    Keeper &k = keeper();
    std::lock_guard<std::mutex> lock(k.mu);
    k.frees += 1;
    while (!k.kept.empty() && (k.kept[0].at + kKeepFrees < k.frees ||
                               (mine.bytes <= kKeepBytes && k.bytes + mine.bytes > kKeepBytes)))
        drop(k, 0);
    if (mine.bytes <= kKeepBytes) {
        try {
            k.kept.push_back(Kept{device, mine, k.frees});
            k.bytes += mine.bytes;
            return;
        } catch (...) {   // no host memory to remember it by
        }
    }
    (void)hipFree(mine.buf);
}

namespace {
// the capture that s takes part in (0: none; the default stream takes part in none)
unsigned long long capture_of(hipStream_t s)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    unsigned long long id = 0;
    if (!s) return 0;
    if (hipStreamGetCaptureInfo(s, &status, &id) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return status == hipStreamCaptureStatusNone ? 0 : id + 1;
}
}  // namespace

void wrote_store(st_ctx *c, hipStream_t s)
{
    const unsigned long long id = capture_of(s);
    if (id) {
        c->capture = id;
        c->capture_stream = s;
    } else {
        c->store_stream = s;
    }
}

bool second_store_free(const st_ctx *c, hipStream_t s)
{
    const unsigned long long id = capture_of(s);
    return id ? id == c->capture && s == c->capture_stream : s == c->store_stream;
}

bool saved_fit(const st_ctx *c, int64_t n)
{
    const size_t left = c->saved_max > c->saved_bytes ? c->saved_max - c->saved_bytes : 0;
    return (int64_t)(c->saved_spare.size() + left / snapshot_bytes(c)) >= n;
}

Block take_saved(st_ctx *c)
{
    Block b;
    if (!c->saved_spare.empty()) {
        b = c->saved_spare.back();
        c->saved_spare.pop_back();
    } else if (saved_fit(c, 1)) {
        if (block_alloc(c->device, snapshot_bytes(c), &b) == hipSuccess) {
            c->saved_bytes += b.bytes;
        } else {
            c->saved_max = c->saved_bytes;   // no more than there are
        }
    }
    return b;
}

void untake_saved(st_ctx *c, size_t n)
{
    for (size_t k = c->saved.size() - n; k < c->saved.size(); ++k) {
        if (c->saved[k].buf) c->saved_spare.push_back(c->saved[k]);
        c->saved[k] = Block{};
    }
}

bool drop_saved(st_ctx *c)
{
    c->saved_max = 0;
    const bool any = c->saved_bytes > 0;
    if (!any || hipDeviceSynchronize() != hipSuccess) return false;
    for (auto *v : {&c->saved, &c->saved_spare})
        for (auto &b : *v) block_free(c->device, &b);
    c->saved_spare.clear();
    c->saved_bytes = 0;
    return true;
}

}  // namespace st

namespace {

constexpr double kPi = 3.14159265358979323846;

// message of the last failed st_create_mesh on this thread (no context yet)
thread_local std::string g_create_err;

st_status fail(st_ctx *c, st_status s, const std::string &msg)
{
    if (c) c->err = msg;
    return s;
}

st_status dev_fail(st_ctx *c, hipError_t e, const char *what)
{
    return fail(c, ST_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

#define ST_HIP(call)                                        \
    do {                                                    \
        hipError_t e_ = (call);                             \
        if (e_ != hipSuccess) return dev_fail(c, e_, #call); \
    } while (0)

// A context's buffers up to this much are one block (each array at 256 bytes,
// large ones at 2 MiB, as separate allocations start); larger contexts live
// long, and are allocated array by array.
constexpr size_t kOneBlock = (size_t)4 << 30;

struct Wanted {
    void **ptr;
    size_t bytes;
};

hipError_t allocate(st_ctx *c, const std::vector<Wanted> &want, size_t &total)
{
    constexpr size_t kLarge = (size_t)2 << 20;
    size_t at = 0;
    std::vector<size_t> off;
    for (const Wanted &w : want) {
        const size_t align = w.bytes >= kLarge ? kLarge : 256;
        at = (at + align - 1) / align * align;
        off.push_back(at);
        at += w.bytes ? w.bytes : 8;
    }
    total = at;
    const bool one = at <= kOneBlock;
    c->blocks.reserve(one ? 1 : want.size());
    for (size_t k = 0; k < (one ? 1 : want.size()); ++k) {
        st::Block b;
        const hipError_t e = st::block_alloc(c->device, one ? at : want[k].bytes, &b);
        if (e != hipSuccess) return e;
        c->blocks.push_back(b);
        *want[k].ptr = b.buf;
    }
    if (one)
        for (size_t k = 0; k < want.size(); ++k) *want[k].ptr = (char *)c->blocks[0].buf + off[k];
    return hipSuccess;
}

void free_all(st_ctx *c)
{
    for (auto *v : {&c->blocks, &c->snaps, &c->spare, &c->saved, &c->saved_spare}) {
        for (auto &b : *v) st::block_free(c->device, &b);
        v->clear();
    }
    st::block_free(c->device, &c->stage64);
    st::block_free(c->device, &c->bwd_ws);
    void *singles[] = {c->fieldbuf[0], c->fieldbuf[1], c->ec_prev, c->ec_ext};
    for (void *p : singles) (void)hipFree(p);
    for (hipEvent_t e : c->tev) (void)hipEventDestroy(e);
    c->tev.clear();
    if (c->side) (void)hipStreamDestroy(c->side);
}

st_status ensure_flushed(st_ctx *c, hipStream_t s)
{
    if (c->pending == 0) return ST_OK;
    ST_HIP(st::launch_flush_pending(c, s));
    c->count += c->pending;
    c->pending = 0;
    return ST_OK;
}

// Device memory that the kept states of taped steps make room for: a buffer for
// one more checkpoint, and a call's temporary or a context's later buffer (for
// hipFree).
hipError_t alloc_checkpoint(st_ctx *c, st::Snapshot *sn)
{
    hipError_t e = st::block_alloc(c->device, st::snapshot_bytes(c), sn);
    if (e == hipErrorOutOfMemory && st::drop_saved(c))
        e = st::block_alloc(c->device, st::snapshot_bytes(c), sn);
    return e;
}

template <class P>
hipError_t alloc(st_ctx *c, P **p, size_t bytes)
{
    hipError_t e = st::device_malloc((void **)p, bytes);
    if (e == hipErrorOutOfMemory && st::drop_saved(c)) e = st::device_malloc((void **)p, bytes);
    return e;
}

bool finite3(const double *v)
{
    return isfinite(v[0]) && isfinite(v[1]) && isfinite(v[2]);
}

}  // namespace

extern "C" {

st_status st_create_mesh(const st_mesh_desc *desc, int device, st_ctx **out)
{
    if (!desc || !out) return ST_ERR_INVALID;
    *out = nullptr;
    st_ctx *c = nullptr;
    try {
        c = new st_ctx();
    } catch (...) {
        return ST_ERR_OOM;
    }
    auto bad = [&](const std::string &m) {
        delete c;
        g_create_err = "st_create_mesh: " + m;
        return ST_ERR_INVALID;
    };
    const st_mesh_desc &d = *desc;
    const int E = d.chunk_edge;
    if (!(E == 2 || E == 4 || E == 8)) return bad("chunk_edge must be 2, 4 or 8");
    for (int a = 0; a < 3; ++a) {
        if (d.n[a] < E || d.n[a] % E != 0) return bad("n must be a positive multiple of chunk_edge");
        if (!(isfinite(d.L[a]) && d.L[a] > 0)) return bad("L must be finite and > 0");
        if (!isfinite(d.g[a])) return bad("g must be finite");
    }
    if (!(isfinite(d.mu_f) && d.mu_f > 0) || !(isfinite(d.rho_p) && d.rho_p > 0) ||
        !(isfinite(d.parcel_weight) && d.parcel_weight > 0) || !isfinite(d.rho_f))
        return bad("material constants must be finite and > 0");
    if (d.form < 0 || d.form > 2) return bad("unknown form");
    if (d.interp < 0 || d.interp > 1) return bad("unknown interpolation");
    if (d.drag < 0 || d.drag > 1) return bad("unknown drag law");
    if (d.reserved != 0) return bad("reserved must be 0");
    if (d.drag == ST_DRAG_SCHILLER_NAUMANN && !(d.rho_f >= 0))
        return bad("rho_f must be >= 0 for Schiller-Naumann drag");
    if (d.capacity < 1) return bad("capacity must be >= 1");
    const int64_t ncell = (int64_t)d.n[0] * d.n[1] * d.n[2];
    if (ncell > ((int64_t)1 << 34)) return bad("mesh too large");

    c->desc = d;
    c->device = device;
    c->form = d.form;
    c->tsize = d.form == ST_FORM_FP64 ? 8 : 4;
    c->asize = d.form == ST_FORM_FP32 ? 4 : 8;
    st::Params &p = c->prm;
    memset(&p, 0, sizeof p);
    p.E = E;
    p.interp = d.interp;
    p.drag = d.drag;
    for (int a = 0; a < 3; ++a) {
        p.n[a] = d.n[a];
        p.nc[a] = d.n[a] / E;
        p.L[a] = d.L[a];
        p.h[a] = d.L[a] / d.n[a];
        p.inv_h[a] = 1.0 / p.h[a];
        p.g[a] = d.g[a];
    }
    p.global = d.form == ST_FORM_FP32 ? 1 : 0;
    for (int a = 0; a < 3; ++a) {
        p.inv_hf[a] = (float)(d.n[a] / d.L[a]);
        p.Lf[a] = (float)d.L[a];
    }
    p.C = (int64_t)p.nc[0] * p.nc[1] * p.nc[2];
    p.inv_V = 1.0 / (p.h[0] * p.h[1] * p.h[2]);
    p.tau_coef = d.rho_p / (18.0 * d.mu_f);
    p.mass_coef = d.parcel_weight * d.rho_p * kPi / 6.0;
    p.re_coef = d.rho_f / d.mu_f;

    c->C = p.C;
    c->cap = d.capacity;
    // containers: one per chunk and one more per kSeg particles (rounded up to
    // the step's launch grid)
    c->max_items = p.C + (d.capacity + st::kSeg - 1) / st::kSeg;
    // spare slots: a quarter of the capacity (at least kSlackMin per chunk),
    // plus what rounding every room up to kAlign can take
    c->slots = d.capacity + std::max<int64_t>(d.capacity / 4, (int64_t)st::kSlackMin * p.C) +
               (int64_t)st::kAlign * c->max_items;
    if (c->slots >= ((int64_t)1 << 31) - 1 || c->max_items >= ((int64_t)1 << 30))
        return bad("capacity too large for 32-bit slot indices");

    auto dev_bad = [&](st_status st, const std::string &m) {
        (void)hipDeviceSynchronize();
        free_all(c);
        delete c;
        g_create_err = "st_create_mesh: " + m;
        return st;
    };
    hipError_t e = hipSetDevice(device);
    if (e != hipSuccess) return dev_bad(ST_ERR_DEVICE, hipGetErrorString(e));
    size_t total = 0;
    const int64_t C = p.C;
    auto stagger = [](int b, int k) { return (size_t)(8 * b + k) * st::kStagger; };
    // The inboxes, and the staging area of injections into a store that holds
    // particles (a full re-bin places them, so a load should fill it few times).
    // Where these do not fit beside the store, smaller ones: the steps then take
    // the full re-bin more often.
    const st::InboxRule rules[3] = {c->slots <= (1 << 17) ? st::InboxRule{0, 0}
                                                          : st::InboxRule{3, 16},
                                    {3, 4}, {5, 0}};
    auto sizes = [&](int level) {
        c->inbox = rules[level];
        c->nrec = (c->slots >> c->inbox.shift) + c->inbox.plus * c->max_items;
        const int64_t stage = level ? std::max<int64_t>(1 << 16, d.capacity / 8)
                                    : std::max<int64_t>(1 << 17, d.capacity / 3 + 1);
        c->mcap = std::min<int64_t>(d.capacity, stage);
        c->staged_stride = level ? 1 : 16;
    };
    hipError_t ok = hipErrorOutOfMemory;
    try {
        const size_t rec = c->tsize == 8 ? sizeof(st::MoverRec<double>)
                                         : sizeof(st::MoverRec<float>);
        for (int level = 0; level < 3 && ok == hipErrorOutOfMemory; ++level) {
            for (auto &b : c->blocks) st::block_free(device, &b);
            c->blocks.clear();
            sizes(level);
            std::vector<Wanted> want;
            auto A = [&](auto **ptr, size_t bytes) { want.push_back({(void **)ptr, bytes}); };
            for (int b = 0; b < 2; ++b)
                for (int k = 0; k < 8; ++k)
                    A(&c->store[b][k], (size_t)c->slots * (k < 7 ? c->tsize : 4) + stagger(b, k));
            for (int b = 0; b < 2; ++b) {
                A(&c->cont[b], (size_t)c->max_items * sizeof(st::Cont));
                A(&c->first[b], (size_t)(C + 1) * 4);
            }
            A(&c->rec, (size_t)(2 * c->nrec) * rec);
            A(&c->stage, (size_t)c->mcap * rec);
            A(&c->stage_dest, (size_t)c->mcap * 4);
            A(&c->staged, (size_t)(C * c->staged_stride) * 4);
            A(&c->cursor, (size_t)C * 4);
            A(&c->new_cnt, (size_t)C * 4);
            A(&c->lay, (size_t)C * 16);
            A(&c->lay_sums, 16);
            A(&c->lay_part, (size_t)(C / 1024 + 1) * 16);
            A(&c->flags, (size_t)st::F_COUNT * 4);
            A(&c->spread, (size_t)st::kSpreadInts * 4);
            A(&c->src, (size_t)3 * ncell * c->asize);
            A(&c->written, (size_t)C * 4);
            ok = allocate(c, want, total);
        }
    } catch (...) {   // host memory
        ok = hipErrorOutOfMemory;
    }
    if (ok != hipSuccess)
        return dev_bad(ST_ERR_OOM, "device allocation of " + std::to_string(total) +
                                       " bytes failed");
    for (int b = 0; b < 2; ++b)
        for (int k = 0; k < 8; ++k) c->store[b][k] = (char *)c->store[b][k] + stagger(b, k);
    // this device's address of the fixed scratch of st_bounding_boxes_noalloc
    e = st::noalloc_scratch_init(device);
    if (e != hipSuccess) return dev_bad(ST_ERR_DEVICE, hipGetErrorString(e));
    hipStream_t s = nullptr;
    e = st::launch_init(c, s);
    if (e == hipSuccess) e = st::launch_zero_sources(c, s);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) return dev_bad(ST_ERR_DEVICE, hipGetErrorString(e));
    *out = c;
    return ST_OK;
}

st_status st_destroy(st_ctx *c)
{
    if (!c) return ST_ERR_INVALID;
    (void)hipSetDevice(c->device);
    (void)hipDeviceSynchronize();
    free_all(c);
    delete c;
    return ST_OK;
}

st_status st_release_memory(void)
{
    try {
        st::release_kept();
        return ST_OK;
    } catch (...) {
        return ST_ERR_DEVICE;
    }
}

const char *st_last_error(const st_ctx *c)
{
    if (!c) return g_create_err.c_str();
    return c->err.c_str();
}

st_status st_count(const st_ctx *c, int64_t *n)
{
    if (!c || !n) return ST_ERR_INVALID;
    *n = c->count + c->pending;
    return ST_OK;
}

st_status st_inject(st_ctx *c, int64_t n, const double *x, const double *up, const double *d,
                    int on_device, void *hip_stream)
{
    if (!c) return ST_ERR_INVALID;
    try {
        if (n < 0) return fail(c, ST_ERR_INVALID, "st_inject: n < 0");
        if (n == 0) return ST_OK;
        if (!x || !up || !d) return fail(c, ST_ERR_INVALID, "st_inject: null array");
        if (c->count + c->pending + n > c->cap)
            return fail(c, ST_ERR_CAPACITY, "st_inject: capacity exceeded");
        if (!c->tape.empty()) return fail(c, ST_ERR_STATE, "st_inject: a tape is recorded");
        if (!on_device) {
            for (int64_t i = 0; i < n; ++i)
                if (!finite3(x + 3 * i) || !finite3(up + 3 * i) || !isfinite(d[i]) || !(d[i] > 0))
                    return fail(c, ST_ERR_INVALID, "st_inject: non-finite value or d <= 0 at " +
                                                       std::to_string(i));
        }
        ST_HIP(hipSetDevice(c->device));
        hipStream_t s = (hipStream_t)hip_stream;
        if (on_device) {
            ST_HIP(st::launch_zero_i32(c->flags + st::F_BADINPUT, 1, s));
        }
        // staged in the store while it is empty
        if (c->pending == 0) c->stage_in_store = c->count == 0;
        const int64_t stage_batch = std::min<int64_t>(c->mcap, 1 << 22);
        if (!on_device && !c->stage64.buf) {
            size_t bytes = (size_t)stage_batch * 7 * 8;
            hipError_t e = st::block_alloc(c->device, bytes, &c->stage64);
            if (e == hipErrorOutOfMemory && st::drop_saved(c))
                e = st::block_alloc(c->device, bytes, &c->stage64);
            if (e != hipSuccess) return fail(c, ST_ERR_OOM, "st_inject: staging buffer");
        }
        const int64_t pend0 = c->pending, id0 = c->next_id, count0 = c->count;
        int64_t done = 0;
        while (done < n) {
            // (an empty store's 7 slots / 8 records are more than the capacity)
            int64_t room = c->stage_in_store ? c->slots / 8 * 7 : c->mcap;
            if (c->pending >= room) {
                st_status r = ensure_flushed(c, s);
                if (r != ST_OK) return r;
                c->stage_in_store = 0;
                room = c->mcap;
            }
            int64_t k = std::min<int64_t>(n - done, room - c->pending);
            if (!on_device) k = std::min<int64_t>(k, stage_batch);
            const double *xs = x + 3 * done, *us = up + 3 * done, *ds = d + done;
            if (!on_device) {
                double *sx = (double *)c->stage64.buf, *su = sx + 3 * stage_batch, *sd = su + 3 * stage_batch;
                ST_HIP(hipMemcpyAsync(sx, xs, (size_t)k * 24, hipMemcpyHostToDevice, s));
                ST_HIP(hipMemcpyAsync(su, us, (size_t)k * 24, hipMemcpyHostToDevice, s));
                ST_HIP(hipMemcpyAsync(sd, ds, (size_t)k * 8, hipMemcpyHostToDevice, s));
                xs = sx;
                us = su;
                ds = sd;
            }
            ST_HIP(st::launch_stage_inject(c, k, xs, us, ds, c->pending, s));
            if (!on_device) ST_HIP(hipStreamSynchronize(s));
            c->pending += k;
            c->next_id += k;
            done += k;
        }
        if (on_device) {
            int32_t badflag = 0;
            ST_HIP(hipMemcpyAsync(&badflag, c->flags + st::F_BADINPUT, 4, hipMemcpyDeviceToHost, s));
            ST_HIP(hipStreamSynchronize(s));
            if (badflag) {
                // undone when no flush happened in between; otherwise the store
                // already holds the batch, its bad droplets left out
                if (c->count == count0) {
                    ST_HIP(st::launch_unstage(c, pend0, s));
                    c->pending = pend0;
                    c->next_id = id0;
                    return fail(c, ST_ERR_INVALID, "st_inject: non-finite value or d <= 0");
                }
                return fail(c, ST_ERR_INVALID,
                            "st_inject: non-finite value or d <= 0 (partially injected)");
            }
        }
        // no more than the staging area holds is left for the next call to place
        if (c->stage_in_store && c->pending > c->mcap) return ensure_flushed(c, s);
        return ST_OK;
    } catch (...) {
        return fail(c, ST_ERR_OOM, "st_inject: host allocation failed");
    }
}

st_status st_step(st_ctx *c, const void *u_cells, double dt, int32_t nsub, int32_t tape,
                  void *hip_stream)
{
    if (!c) return ST_ERR_INVALID;
    try {
        if (!u_cells) return fail(c, ST_ERR_INVALID, "st_step: null field");
        if (!(isfinite(dt) && dt > 0)) return fail(c, ST_ERR_INVALID, "st_step: dt must be finite and > 0");
        if (nsub < 1) return fail(c, ST_ERR_INVALID, "st_step: nsub must be >= 1");
        if (tape < 0) return fail(c, ST_ERR_INVALID, "st_step: tape must be >= 0");
        if (tape > 0 && c->form == ST_FORM_FP32)
            return fail(c, ST_ERR_INVALID,
                        "st_step: taped steps need the FP64 or FP32 chunk-local form");
        if (tape > 0 && c->tape.empty() && c->tape_every == 0) c->tape_every = tape;
        if (tape == 0 && !c->tape.empty())
            return fail(c, ST_ERR_STATE, "st_step: untaped step while a tape is recorded");
        ST_HIP(hipSetDevice(c->device));
        hipStream_t s = (hipStream_t)hip_stream;
        st_status r = ensure_flushed(c, s);
        if (r != ST_OK) return r;
        const double dts = dt / nsub;
        for (int32_t k = 0; k < nsub; ++k) {
            if (tape > 0) {
                st::Block state;   // the step's, for the reverse
                const size_t pos = c->tape.size() % (size_t)c->tape_every;
                if (pos == 0) {
                    st::Snapshot sn;
                    if (!c->spare.empty()) {   // a buffer of a consumed tape
                        sn = c->spare.back();
                        c->spare.pop_back();
                    } else {
                        if (alloc_checkpoint(c, &sn) != hipSuccess)
                            return fail(c, ST_ERR_OOM, "st_step: checkpoint");
                    }
                    c->snaps.push_back(sn);
                    ST_HIP(st::launch_snapshot(c, sn.buf, 0, s));
                } else if (pos == 1 ? st::saved_fit(c, c->tape_every - 1)
                                    : c->saved.back().buf != nullptr) {
                    // a segment's states are kept if all of them fit: one
                    // that lacks some is recomputed whole
                    state = st::take_saved(c);
                    if (!state.buf) st::untake_saved(c, pos - 1);
                }
                c->saved.push_back(state);
                c->tape.push_back(st::TapeStep{u_cells, dts});
                ST_HIP(st::launch_step(c, u_cells, dts, 1, s, state.buf));
                continue;
            }
            ST_HIP(st::launch_step(c, u_cells, dts, 1, s));
        }
        return ST_OK;
    } catch (...) {
        return fail(c, ST_ERR_OOM, "st_step: host allocation failed");
    }
}

st_status st_get_sources(st_ctx *c, double *out, int32_t reset, int on_device, void *hip_stream)
{
    if (!c) return ST_ERR_INVALID;
    if (!out) return fail(c, ST_ERR_INVALID, "st_get_sources: null output");
    ST_HIP(hipSetDevice(c->device));
    hipStream_t s = (hipStream_t)hip_stream;
    const size_t n = 3 * (size_t)c->prm.n[0] * c->prm.n[1] * c->prm.n[2];
    if (on_device) {
        ST_HIP(st::launch_get_sources(c, out, reset, s));
        return ST_OK;
    }
    double *tmp = nullptr;
    hipError_t e = alloc(c, &tmp, n * 8);
    if (e != hipSuccess) return fail(c, ST_ERR_OOM, "st_get_sources: temporary");
    e = st::launch_get_sources(c, tmp, reset, s);
    if (e == hipSuccess) e = hipMemcpyAsync(out, tmp, n * 8, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipFree(tmp);
    if (e != hipSuccess) return dev_fail(c, e, "st_get_sources");
    return ST_OK;
}

st_status st_get_particles(st_ctx *c, double *x, double *up, double *d, int64_t *id,
                           int32_t *cell, int on_device, void *hip_stream)
{
    if (!c) return ST_ERR_INVALID;
    ST_HIP(hipSetDevice(c->device));
    hipStream_t s = (hipStream_t)hip_stream;
    st_status r = ensure_flushed(c, s);
    if (r != ST_OK) return r;
    const size_t n = (size_t)c->count;
    if (on_device) {
        ST_HIP(st::launch_get_particles(c, x, up, d, id, cell, s));
        return ST_OK;
    }
    if (n == 0) return ST_OK;
    // one device temporary laid out as x, up, d, id, cell
    size_t bytes = n * (24 + 24 + 8 + 8 + 12);
    char *tmp = nullptr;
    hipError_t e = alloc(c, &tmp, bytes);
    if (e != hipSuccess) return fail(c, ST_ERR_OOM, "st_get_particles: temporary");
    double *tx = (double *)tmp, *tu = tx + 3 * n, *td = tu + 3 * n;
    int64_t *ti = (int64_t *)(td + n);
    int32_t *tc = (int32_t *)(ti + n);
    e = st::launch_get_particles(c, x ? tx : nullptr, up ? tu : nullptr, d ? td : nullptr,
                                 id ? ti : nullptr, cell ? tc : nullptr, s);
    if (e == hipSuccess && x) e = hipMemcpyAsync(x, tx, n * 24, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess && up) e = hipMemcpyAsync(up, tu, n * 24, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess && d) e = hipMemcpyAsync(d, td, n * 8, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess && id) e = hipMemcpyAsync(id, ti, n * 8, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess && cell) e = hipMemcpyAsync(cell, tc, n * 12, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipFree(tmp);
    if (e != hipSuccess) return dev_fail(c, e, "st_get_particles");
    return ST_OK;
}

namespace {

// Drops the tape; its checkpoint buffers are kept for the next tape, or
// released with the backward workspace.
void tape_reset(st_ctx *c, bool keep_buffers)
{
    (void)hipSetDevice(c->device);
    (void)hipDeviceSynchronize();
    for (auto &sn : c->snaps) {
        if (keep_buffers) c->spare.push_back(sn);
        else st::block_free(c->device, &sn);
    }
    c->snaps.clear();
    if (!keep_buffers) {
        for (auto &sn : c->spare) st::block_free(c->device, &sn);
        c->spare.clear();
        st::block_free(c->device, &c->bwd_ws);
    }
    for (auto &b : c->saved)
        if (b.buf) c->saved_spare.push_back(b);
    c->saved.clear();
    if (!keep_buffers) {
        (void)st::drop_saved(c);
        c->saved_max = st::kSavedBytes;
    }
    c->tape.clear();
    c->tape_every = 0;
}

}  // namespace

st_status st_tape_clear(st_ctx *c)
{
    if (!c) return ST_ERR_INVALID;
    try {
        tape_reset(c, false);
        return ST_OK;
    } catch (...) {
        return fail(c, ST_ERR_OOM, "st_tape_clear: host allocation failed");
    }
}

st_status st_tape_reserve(st_ctx *c, int32_t tape, int64_t substeps)
{
    if (!c) return ST_ERR_INVALID;
    if (tape <= 0 || substeps < 0)
        return fail(c, ST_ERR_INVALID, "st_tape_reserve: tape must be > 0 and substeps >= 0");
    if (c->form == ST_FORM_FP32)
        return fail(c, ST_ERR_INVALID,
                    "st_tape_reserve: taped steps need the FP64 or FP32 chunk-local form");
    if (!c->tape.empty()) return fail(c, ST_ERR_STATE, "st_tape_reserve: a tape is recorded");
    try {
        ST_HIP(hipSetDevice(c->device));
        const int64_t need = (substeps + tape - 1) / tape;
        while ((int64_t)c->spare.size() < need) {
            st::Snapshot sn;
            if (alloc_checkpoint(c, &sn) != hipSuccess)
                return fail(c, ST_ERR_OOM, "st_tape_reserve: checkpoint");
            c->spare.push_back(sn);
        }
        // the states of the steps between the checkpoints, for the segments that
        // the run will keep them for
        int64_t states = 0;
        auto kept = [&]() {   // (whether that is all of them)
            states = 0;
            for (int64_t left = substeps; left > 0; left -= tape) {
                const int64_t n = std::min<int64_t>(left, tape) - 1;
                if (n > 0 && !st::saved_fit(c, states + tape - 1)) return false;
                states += n;
            }
            return true;
        };
        bool all = kept();
        while ((int64_t)c->saved_spare.size() < states) {
            c->saved_spare.reserve(c->saved_spare.size() + 1);
            std::vector<st::Block> held;
            held.swap(c->saved_spare);
            const st::Block b = st::take_saved(c);
            held.swap(c->saved_spare);
            if (b.buf) c->saved_spare.push_back(b);
            else all = kept();   // fewer than they were to be
        }
        // they are given up where they leave no room for the rest
        hipError_t e = st::reserve_backward(c, tape, !all);
        if (e == hipErrorOutOfMemory && st::drop_saved(c))
            e = st::reserve_backward(c, tape, substeps > need);
        if (e != hipSuccess) return fail(c, ST_ERR_OOM, "st_tape_reserve: backward workspace");
        return ST_OK;
    } catch (...) {
        return fail(c, ST_ERR_OOM, "st_tape_reserve: host allocation failed");
    }
}

st_status st_backward(st_ctx *c, const double *dL_dSint, double *dL_du, double *dL_dd,
                      void *hip_stream)
{
    if (!c) return ST_ERR_INVALID;
    if (!dL_dSint || !dL_du || (!dL_dd && c->count > 0))
        return fail(c, ST_ERR_INVALID, "st_backward: null pointer");
    if (c->tape.empty()) return fail(c, ST_ERR_STATE, "st_backward: nothing taped");
    ST_HIP(hipSetDevice(c->device));
    try {
        ST_HIP(st::launch_backward(c, dL_dSint, dL_du, dL_dd, (hipStream_t)hip_stream));
        tape_reset(c, true);
        return ST_OK;
    } catch (...) {
        return fail(c, ST_ERR_OOM, "st_backward: host allocation failed");
    }
}

st_status st_run_coupled(st_ctx *c, const void *u0, const double *cs, int32_t nsteps, double dt,
                         float *field_ms, float *step_ms, float *total_ms, void *hip_stream)
{
    if (!c) return ST_ERR_INVALID;
    if (!u0 || !cs) return fail(c, ST_ERR_INVALID, "st_run_coupled: null pointer");
    if (nsteps < 0) return fail(c, ST_ERR_INVALID, "st_run_coupled: nsteps < 0");
    if (!(isfinite(dt) && dt > 0)) return fail(c, ST_ERR_INVALID, "st_run_coupled: bad dt");
    if (!c->tape.empty()) return fail(c, ST_ERR_STATE, "st_run_coupled: a tape is recorded");
    for (int32_t k = 0; k < nsteps; ++k)
        if (!isfinite(cs[2 * k]) || !isfinite(cs[2 * k + 1]))
            return fail(c, ST_ERR_INVALID, "st_run_coupled: non-finite rotation");
    if (nsteps == 0) return ST_OK;
    ST_HIP(hipSetDevice(c->device));
    hipStream_t sa = (hipStream_t)hip_stream;
    st_status r = ensure_flushed(c, sa);
    if (r != ST_OK) return r;
    const size_t fbytes = 3 * (size_t)c->prm.n[0] * c->prm.n[1] * c->prm.n[2] * c->tsize;
    for (int b = 0; b < 2; ++b)
        if (!c->fieldbuf[b]) {
            hipError_t e = alloc(c, &c->fieldbuf[b], fbytes);
            if (e != hipSuccess) return fail(c, ST_ERR_OOM, "st_run_coupled: field buffers");
        }
    if (!c->side) ST_HIP(hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking));
    hipStream_t sb = c->side;
    const bool timed = field_ms || step_ms || total_ms;
    // events: field k ready, step k done (its field buffer may be reused)
    std::vector<hipEvent_t> ev_field(nsteps), ev_step(nsteps);
    std::vector<hipEvent_t> tf0(nsteps), tf1(nsteps), ts0(nsteps), ts1(nsteps);
    hipEvent_t t_begin = nullptr, t_end = nullptr;
    auto cleanup = [&]() {
        for (auto *v : {&ev_field, &ev_step, &tf0, &tf1, &ts0, &ts1})
            for (hipEvent_t e : *v)
                if (e) (void)hipEventDestroy(e);
        if (t_begin) (void)hipEventDestroy(t_begin);
        if (t_end) (void)hipEventDestroy(t_end);
    };
    hipError_t e = hipSuccess;
    for (int32_t k = 0; k < nsteps && e == hipSuccess; ++k) {
        e = hipEventCreateWithFlags(&ev_field[k], hipEventDisableTiming);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&ev_step[k], hipEventDisableTiming);
        if (timed) {
            if (e == hipSuccess) e = hipEventCreate(&tf0[k]);
            if (e == hipSuccess) e = hipEventCreate(&tf1[k]);
            if (e == hipSuccess) e = hipEventCreate(&ts0[k]);
            if (e == hipSuccess) e = hipEventCreate(&ts1[k]);
        }
    }
    if (e == hipSuccess && timed) e = hipEventCreate(&t_begin);
    if (e == hipSuccess && timed) e = hipEventCreate(&t_end);
    // the side stream starts after everything already on the caller's stream
    hipEvent_t ev_start = nullptr;
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ev_start, hipEventDisableTiming);
    if (e == hipSuccess && timed) e = hipEventRecord(t_begin, sa);
    if (e == hipSuccess) e = hipEventRecord(ev_start, sa);
    if (e == hipSuccess) e = hipStreamWaitEvent(sb, ev_start, 0);
    // field 0 first
    for (int32_t k = 0; k <= nsteps && e == hipSuccess; ++k) {
        // stream B: build U^(k) ... lagging the particle stream by one step
        if (k < nsteps) {
            void *buf = c->fieldbuf[k & 1];
            if (k >= 2) e = hipStreamWaitEvent(sb, ev_step[k - 2], 0);  // buffer free again
            if (e == hipSuccess && timed) e = hipEventRecord(tf0[k], sb);
            if (e == hipSuccess) e = st::launch_rotate_field(c, u0, buf, cs[2 * k], cs[2 * k + 1], sb);
            if (e == hipSuccess && timed) e = hipEventRecord(tf1[k], sb);
            if (e == hipSuccess) e = hipEventRecord(ev_field[k], sb);
        }
        // stream A: step k-1 with U^(k-1) while U^(k) is being built
        if (k >= 1 && e == hipSuccess) {
            const int32_t j = k - 1;
            e = hipStreamWaitEvent(sa, ev_field[j], 0);
            if (e == hipSuccess && timed) e = hipEventRecord(ts0[j], sa);
            if (e == hipSuccess) e = st::launch_step(c, c->fieldbuf[j & 1], dt, 1, sa);
            if (e == hipSuccess && timed) e = hipEventRecord(ts1[j], sa);
            if (e == hipSuccess) e = hipEventRecord(ev_step[j], sa);
        }
    }
    // the caller's stream must not run ahead of the side stream
    if (e == hipSuccess) e = hipEventRecord(ev_start, sb);
    if (e == hipSuccess) e = hipStreamWaitEvent(sa, ev_start, 0);
    if (e == hipSuccess && timed) e = hipEventRecord(t_end, sa);
    if (e == hipSuccess && timed) e = hipEventSynchronize(t_end);
    if (e == hipSuccess && timed) {
        float fsum = 0, ssum = 0, ms = 0;
        for (int32_t k = 0; k < nsteps && e == hipSuccess; ++k) {
            e = hipEventElapsedTime(&ms, tf0[k], tf1[k]);
            fsum += ms;
            if (e == hipSuccess) e = hipEventElapsedTime(&ms, ts0[k], ts1[k]);
            ssum += ms;
        }
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, t_begin, t_end);
        if (field_ms) *field_ms = fsum;
        if (step_ms) *step_ms = ssum;
        if (total_ms) *total_ms = ms;
    }
    if (!timed && e == hipSuccess) e = hipStreamSynchronize(sa);
    if (ev_start) (void)hipEventDestroy(ev_start);
    cleanup();
    if (e != hipSuccess) return dev_fail(c, e, "st_run_coupled");
    return ST_OK;
}

st_status st_ec_reset(st_ctx *c, void *hip_stream)
{
    if (!c) return ST_ERR_INVALID;
    ST_HIP(hipSetDevice(c->device));
    hipStream_t s = (hipStream_t)hip_stream;
    const int64_t n = 3 * (int64_t)c->prm.n[0] * c->prm.n[1] * c->prm.n[2];
    if (!c->ec_prev) {
        if (alloc(c, &c->ec_prev, (size_t)n * 8) != hipSuccess)
            return fail(c, ST_ERR_OOM, "st_ec_reset: history buffers");
        if (alloc(c, &c->ec_ext, (size_t)n * 8) != hipSuccess) {
            (void)hipFree(c->ec_prev);
            c->ec_prev = nullptr;
            return fail(c, ST_ERR_OOM, "st_ec_reset: history buffers");
        }
    }
    ST_HIP(st::launch_zero_f64(c->ec_prev, n, s));
    ST_HIP(st::launch_zero_f64(c->ec_ext, n, s));
    return ST_OK;
}

st_status st_ec_estimate(st_ctx *c, int32_t kind, const double *S_last, double *applied,
                         int on_device, void *hip_stream)
{
    if (!c) return ST_ERR_INVALID;
    if (!S_last || !applied) return fail(c, ST_ERR_INVALID, "st_ec_estimate: null array");
    if (kind < ST_EXTRAP_ZERO || kind > ST_EXTRAP_LINEAR)
        return fail(c, ST_ERR_INVALID, "st_ec_estimate: unknown extrapolator");
    if (!c->ec_prev) {
        st_status r = st_ec_reset(c, hip_stream);
        if (r != ST_OK) return r;
    }
    ST_HIP(hipSetDevice(c->device));
    hipStream_t s = (hipStream_t)hip_stream;
    const size_t n = 3 * (size_t)c->prm.n[0] * c->prm.n[1] * c->prm.n[2];
    if (on_device) {
        ST_HIP(st::launch_ec(c, kind, S_last, applied, s));
        return ST_OK;
    }
    double *tmp = nullptr;
    if (alloc(c, &tmp, 2 * n * 8) != hipSuccess)
        return fail(c, ST_ERR_OOM, "st_ec_estimate: temporaries");
    hipError_t e = hipMemcpyAsync(tmp, S_last, n * 8, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = st::launch_ec(c, kind, tmp, tmp + n, s);
    if (e == hipSuccess) e = hipMemcpyAsync(applied, tmp + n, n * 8, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipStreamSynchronize(s);
    (void)hipFree(tmp);
    if (e != hipSuccess) return dev_fail(c, e, "st_ec_estimate");
    return ST_OK;
}

st_status st_stats(st_ctx *c, int64_t *last_movers, int64_t *repacks, int64_t *particles,
                   int64_t *slots, int64_t *items, int64_t *holes, void *hip_stream)
{
    if (!c) return ST_ERR_INVALID;
    ST_HIP(hipSetDevice(c->device));
    hipStream_t s = (hipStream_t)hip_stream;
    int32_t f[st::F_COUNT];
    ST_HIP(st::launch_stats(c, s));
    ST_HIP(hipMemcpyAsync(f, c->flags, sizeof f, hipMemcpyDeviceToHost, s));
    ST_HIP(hipStreamSynchronize(s));
    if (last_movers) *last_movers = f[st::F_LASTMOV];
    if (repacks) *repacks = f[st::F_REPACKS];
    if (particles) *particles = c->count + c->pending;
    if (slots) *slots = c->slots;
    if (items) *items = f[st::F_STAT_ITEMS];
    if (holes) *holes = f[st::F_STAT_HOLES];
    return ST_OK;
}

st_status st_stream_copy(const void *src, void *dst, int64_t bytes, void *hip_stream)
{
    if (!src || !dst || bytes < 0 || bytes % 16 != 0 || ((uintptr_t)src | (uintptr_t)dst) % 16)
        return ST_ERR_INVALID;
    if (bytes == 0) return ST_OK;
    return st::launch_stream_copy(src, dst, bytes, (hipStream_t)hip_stream) == hipSuccess
               ? ST_OK : ST_ERR_DEVICE;
}

st_status st_timing(st_ctx *c, int32_t enable, double *kernel_ms, int64_t *launches)
{
    if (!c) return ST_ERR_INVALID;
    ST_HIP(hipSetDevice(c->device));
    double sum = 0.0;
    for (size_t k = 0; k + 1 < c->tev.size(); k += 2) {
        ST_HIP(hipEventSynchronize(c->tev[k + 1]));
        float ms = 0.f;
        ST_HIP(hipEventElapsedTime(&ms, c->tev[k], c->tev[k + 1]));
        sum += ms;
    }
    if (kernel_ms) *kernel_ms = sum;
    if (launches) *launches = (int64_t)(c->tev.size() / 2);
    if (enable) {
        for (hipEvent_t e : c->tev) (void)hipEventDestroy(e);
        c->tev.clear();
    }
    c->timing = enable ? 1 : 0;
    return ST_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Hilbert-segment placement and partition bounding boxes
// ---------------------------------------------------------------------------
namespace {

const char *hilbert_args_error(int32_t order, int64_t nseg, int64_t seg_begin, int64_t seg_end,
                               int64_t per_seg)
{
    if (order < 1 || order > 10) return "order must be 1..10";
    if (nseg < 1 || nseg > ((int64_t)1 << (3 * order))) return "nseg must be 1..8^order";
    if (seg_begin < 0 || seg_end > nseg || seg_begin > seg_end)
        return "need 0 <= seg_begin <= seg_end <= nseg";
    if (per_seg < 1 || per_seg > ((int64_t)1 << 31)) return "per_seg must be 1..2^31";
    return nullptr;
}

}  // namespace

st_status st_hilbert_positions(st_ctx *c, int32_t order, int64_t nseg, int64_t seg_begin,
                               int64_t seg_end, int64_t per_seg, const double *u, double *x,
                               int on_device, void *hip_stream)
{
    if (!c) return ST_ERR_INVALID;
    try {
        if (const char *m = hilbert_args_error(order, nseg, seg_begin, seg_end, per_seg))
            return fail(c, ST_ERR_INVALID, std::string("st_hilbert_positions: ") + m);
        const int64_t n = (seg_end - seg_begin) * per_seg;
        if (n == 0) return ST_OK;
        if (!u || !x) return fail(c, ST_ERR_INVALID, "st_hilbert_positions: null array");
        ST_HIP(hipSetDevice(c->device));
        hipStream_t s = (hipStream_t)hip_stream;
        if (on_device) {
            ST_HIP(st::launch_hilbert_positions(order, nseg, seg_begin, per_seg, c->prm.L, 0, n,
                                                u, x, s));
            return ST_OK;
        }
        double *tmp = nullptr;
        if (alloc(c, &tmp, (size_t)n * 48) != hipSuccess)
            return fail(c, ST_ERR_OOM, "st_hilbert_positions: temporaries");
        hipError_t e = hipMemcpyAsync(tmp, u, (size_t)n * 24, hipMemcpyHostToDevice, s);
        if (e == hipSuccess)
            e = st::launch_hilbert_positions(order, nseg, seg_begin, per_seg, c->prm.L, 0, n, tmp,
                                             tmp + 3 * n, s);
        if (e == hipSuccess)
            e = hipMemcpyAsync(x, tmp + 3 * n, (size_t)n * 24, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        (void)hipStreamSynchronize(s);
        (void)hipFree(tmp);
        if (e != hipSuccess) return dev_fail(c, e, "st_hilbert_positions");
        return ST_OK;
    } catch (...) {
        return fail(c, ST_ERR_OOM, "st_hilbert_positions: host allocation failed");
    }
}

st_status st_inject_hilbert(st_ctx *c, int32_t order, int64_t nseg, int64_t seg_begin,
                            int64_t seg_end, int64_t per_seg, const double *u, const double *up,
                            const double *d, int on_device, void *hip_stream)
{
    if (!c) return ST_ERR_INVALID;
    try {
        if (const char *m = hilbert_args_error(order, nseg, seg_begin, seg_end, per_seg))
            return fail(c, ST_ERR_INVALID, std::string("st_inject_hilbert: ") + m);
        const int64_t n = (seg_end - seg_begin) * per_seg;
        if (n == 0) return ST_OK;
        if (!u || !up || !d) return fail(c, ST_ERR_INVALID, "st_inject_hilbert: null array");
        if (c->count + c->pending + n > c->cap)
            return fail(c, ST_ERR_CAPACITY, "st_inject_hilbert: capacity exceeded");
        if (!c->tape.empty()) return fail(c, ST_ERR_STATE, "st_inject_hilbert: a tape is recorded");
        if (!on_device) {
            for (int64_t i = 0; i < n; ++i) {
                for (int a = 0; a < 3; ++a)
                    if (!(u[3 * i + a] >= 0.0 && u[3 * i + a] < 1.0))
                        return fail(c, ST_ERR_INVALID,
                                    "st_inject_hilbert: u outside [0, 1) at " + std::to_string(i));
                if (!finite3(up + 3 * i) || !isfinite(d[i]) || !(d[i] > 0))
                    return fail(c, ST_ERR_INVALID, "st_inject_hilbert: non-finite value or d <= 0 at " +
                                                       std::to_string(i));
            }
        }
        ST_HIP(hipSetDevice(c->device));
        hipStream_t s = (hipStream_t)hip_stream;
        // positions (and, from the host, the other inputs) in device batches,
        // each injected as device arrays
        const int64_t batch = std::min<int64_t>(n, (int64_t)1 << 22);
        double *tmp = nullptr;
        const size_t per = on_device ? 24 : 24 + 24 + 24 + 8;
        if (alloc(c, &tmp, (size_t)batch * per) != hipSuccess)
            return fail(c, ST_ERR_OOM, "st_inject_hilbert: temporaries");
        st_status r = ST_OK;
        hipError_t e = hipSuccess;
        for (int64_t done = 0; done < n && r == ST_OK && e == hipSuccess; done += batch) {
            const int64_t k = std::min<int64_t>(batch, n - done);
            double *xs = tmp;
            const double *us = u + 3 * done, *vs = up + 3 * done, *ds = d + done;
            if (!on_device) {
                double *tu = tmp + 3 * batch, *tv = tu + 3 * batch, *td = tv + 3 * batch;
                e = hipMemcpyAsync(tu, us, (size_t)k * 24, hipMemcpyHostToDevice, s);
                if (e == hipSuccess) e = hipMemcpyAsync(tv, vs, (size_t)k * 24, hipMemcpyHostToDevice, s);
                if (e == hipSuccess) e = hipMemcpyAsync(td, ds, (size_t)k * 8, hipMemcpyHostToDevice, s);
                us = tu;
                vs = tv;
                ds = td;
            }
            if (e == hipSuccess)
                e = st::launch_hilbert_positions(order, nseg, seg_begin, per_seg, c->prm.L, done, k,
                                                 us, xs, s);
            if (e == hipSuccess) r = st_inject(c, k, xs, vs, ds, 1, hip_stream);
        }
        (void)hipStreamSynchronize(s);
        (void)hipFree(tmp);
        if (e != hipSuccess) return dev_fail(c, e, "st_inject_hilbert");
        return r;
    } catch (...) {
        return fail(c, ST_ERR_OOM, "st_inject_hilbert: host allocation failed");
    }
}

st_status st_bounding_boxes(st_ctx *c, int64_t id0, int64_t per_part, int64_t nparts,
                            double *boxes, int on_device, void *hip_stream)
{
    if (!c) return ST_ERR_INVALID;
    if (!boxes) return fail(c, ST_ERR_INVALID, "st_bounding_boxes: null array");
    if (id0 < 0 || per_part < 1 || nparts < 1)
        return fail(c, ST_ERR_INVALID, "st_bounding_boxes: need id0 >= 0, per_part >= 1, nparts >= 1");
    ST_HIP(hipSetDevice(c->device));
    hipStream_t s = (hipStream_t)hip_stream;
    st_status r = ensure_flushed(c, s);
    if (r != ST_OK) return r;
    if (on_device) {
        ST_HIP(st::launch_bounding_boxes(c, id0, per_part, nparts, boxes, s));
        return ST_OK;
    }
    double *tmp = nullptr;
    if (alloc(c, &tmp, (size_t)nparts * 48) != hipSuccess)
        return fail(c, ST_ERR_OOM, "st_bounding_boxes: temporaries");
    hipError_t e = st::launch_bounding_boxes(c, id0, per_part, nparts, tmp, s);
    if (e == hipSuccess) e = hipMemcpyAsync(boxes, tmp, (size_t)nparts * 48, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipStreamSynchronize(s);
    (void)hipFree(tmp);
    if (e != hipSuccess) return dev_fail(c, e, "st_bounding_boxes");
    return ST_OK;
}

st_status st_bounding_boxes_noalloc(st_ctx *c, int64_t id0, int64_t per_part, int64_t nparts,
                                    double *boxes, int32_t on_device, void *hip_stream)
{
    if (!c) return ST_ERR_INVALID;
    if (!boxes) return fail(c, ST_ERR_INVALID, "st_bounding_boxes_noalloc: null array");
    if (id0 < 0 || per_part < 1 || nparts < 1)
        return fail(c, ST_ERR_INVALID,
                    "st_bounding_boxes_noalloc: need id0 >= 0, per_part >= 1, nparts >= 1");
    if (nparts > st::kNoAllocMaxParts)
        return fail(c, ST_ERR_INVALID, "st_bounding_boxes_noalloc: nparts " +
                                           std::to_string(nparts) + " exceeds the maximum " +
                                           std::to_string(st::kNoAllocMaxParts));
    ST_HIP(hipSetDevice(c->device));
    double *sc = nullptr;
    ST_HIP(st::noalloc_scratch(c->device, &sc));
    hipStream_t s = (hipStream_t)hip_stream;
    st_status r = ensure_flushed(c, s);
    if (r != ST_OK) return r;
    ST_HIP(st::launch_bounding_boxes(c, id0, per_part, nparts, sc, s));
    ST_HIP(hipMemcpyAsync(boxes, sc, (size_t)nparts * 48,
                          on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, s));
    if (!on_device) ST_HIP(hipStreamSynchronize(s));
    return ST_OK;
}
