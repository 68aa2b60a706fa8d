// Internal declarations of the scaletrack HIP library (not part of the ABI).
//
// Particle store: structure of arrays, kept sorted by chunk (a cube of
// E^3 cells, E = chunk_edge).  A chunk's particles lie in one or more
// containers (one per kSeg particles at the last full re-bin): container j
// owns the slot range [base, base + room); its particles sit in the first cnt
// slots of that range, among h holes: slots a particle left (an offset of
// kHoleMark or below in binary32, a negative diameter in binary64) or was in
// when its position ceased to be finite (the offset, in both).  Particles that
// crossed into the chunk in the last step wait as `in` records in the
// container's inbox; the next step's kernel takes them up as it streams the
// container (into the holes, then past the last slot).
// Positions are stored as chunk-local offsets in cell units, xi in [0, E)
// per axis; the chunk origin is exact (the chunk index times E cells).  The
// FP32-everywhere form stores binary32 coordinates in metres instead, and
// takes the cell from their binary32 product with n / L.  A full re-bin
// scatters into a second store, which then becomes the store: the device flag
// F_CUR says which of the two it is, and every kernel gets both stores'
// pointers as arguments (so every access is a global-memory instruction).
// All of the state that a step reads and writes lives on the device (the
// flags, the step's tick), so a captured step can be replayed.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "st.h"

namespace st {

constexpr int kSeg = 16384;       // particles per container at a full re-bin, at most
constexpr int kRoomMax = 32768;   // slots per container, at most
constexpr int kSlackMin = 32;     // spare-slot weight per chunk in the room formula
constexpr int kMoverStage = 384;  // movers per workgroup staged in LDS
constexpr int kPool = 128;        // arrivals per workgroup staged in LDS
constexpr int kAlign = 4;         // container rooms are whole multiples of this
// binary32: an offset at or below this marks a hole
constexpr float kHoleMark = -1e30f;
// The state arrays are streamed together at equal slot indices; array k of
// store b starts (8 b + k) kStagger bytes into its allocation, so that equal
// indices of different arrays do not fall on the same HBM channels (aligned
// starts measured 14 % slower on the 1.4e9-particle plume workload; staggers
// of 1 KiB to 17 KiB all remove it, 256 B does not).
constexpr size_t kStagger = 4096 + 256;
// partitions st_bounding_boxes_noalloc can take (its fixed device scratch)
constexpr int64_t kNoAllocMaxParts = 65536;

template <class T>
struct View {
    T *ox, *oy, *oz;   // chunk-local offsets [cells] (FP32-everywhere form: metres)
    T *vx, *vy, *vz;   // velocity [m/s]
    T *d;              // diameter [m]; binary64: -d marks a hole (the state
                       // of the particle that left it is still in place)
    int32_t *id;       // particle id
};

// The store and the re-bin's target; F_CUR says which is which.
template <class T>
struct Views {
    View<T> a, b;
    __host__ __device__ __forceinline__ View<T> pick(int cur) const
    {
        return View<T>{cur ? b.ox : a.ox, cur ? b.oy : a.oy, cur ? b.oz : a.oz,
                       cur ? b.vx : a.vx, cur ? b.vy : a.vy, cur ? b.vz : a.vz,
                       cur ? b.d : a.d,   cur ? b.id : a.id};
    }
};

// A container: its place, and its state after each of the last three steps,
// by the tick modulo 3.  A step at tick t reads the state t - 1 of its own
// container and of its neighbours, adds its movers to in[t] of theirs, and
// writes cnt[t] and h[t] of its own and the zero of in[t + 1]: no two of
// these are the same words, so a step needs no order among its workgroups.
// 64 bytes, so that one scalar load takes all of it.
struct alignas(64) Cont {
    int32_t c;             // chunk
    int32_t base, room;    // slots
    int32_t ibase;         // first record of its inbox
    int32_t k;             // containers of the chunk
    int32_t in[3];         // records in the inbox (arrivals of the step)
    struct { int32_t cnt, h; } s[3];   // slots in use, holes among them
    int32_t place[2];      // full re-bin: places in the chunk of its particles, its records
};
static_assert(sizeof(Cont) == 64, "a container is one 64-byte line");

// Records an inbox holds (more arrivals in one step take the full re-bin): a
// share of its container's room, 1 / 2^shift, and some.  The whole rooms in a
// small store; else an eighth and 16, which on meshes of many sparse chunks is
// a large part of a context (512^3 cells in chunks of 2^3: 22 GB of 67 in
// binary32); where that does not fit, an eighth and 4, and then a 32nd.  (Not less
// at once: with an eighth and 4, 3e7 droplets in 2 097 152 chunks took a full
// re-bin every step, 33.9 ms a step against 25.6.)
struct InboxRule {
    int32_t shift, plus;
};
__host__ __device__ __forceinline__ int32_t inbox_cap(int32_t room, InboxRule rule)
{
    return (room >> rule.shift) + rule.plus;
}

// One particle in flight between chunks (also staged by st_inject), kept together
// so that moving it reads and writes whole 16-byte vectors: 32 bytes in binary32,
// 64 in binary64.
template <class T>
struct alignas(16) MoverRec {
    T ox, oy, oz, vx, vy, vz, d;
    int32_t id;
};
static_assert(sizeof(MoverRec<float>) == 32, "binary32 mover record is 32 bytes");
static_assert(sizeof(MoverRec<double>) == 64, "binary64 mover record is 64 bytes");

// Scalars of the mesh and material used by the kernels.
struct Params {
    int32_t n[3];          // cells per axis
    int32_t nc[3];         // chunks per axis
    int32_t E;             // chunk edge
    int32_t interp;        // 0 trilinear, 1 nearest grid point
    int32_t drag;          // 0 Stokes, 1 Schiller-Naumann
    int32_t pad_;
    int64_t C;             // chunks
    double L[3];           // domain extent
    double h[3];           // cell widths
    double inv_h[3];
    double inv_V;          // 1 / cell volume
    double g[3];
    double tau_coef;       // rho_p / (18 mu_f): tau = tau_coef d^2
    double mass_coef;      // w rho_p pi / 6:    m = mass_coef d^3
    double re_coef;        // rho_f / mu_f:      Re = re_coef d |u_f - u_p|
    // FP32-everywhere form: positions are stored as binary32 coordinates in
    // metres (global != 0); its cell arithmetic in binary32
    float inv_hf[3];       // binary32 n / L per axis
    float Lf[3];           // binary32 L per axis
    int32_t global;
    int32_t pad2_;
};

// Flags and counters on the device (one int32 each).  F_OVERFLOW: the step
// needs a full re-bin; F_FORCE: so does the next one; F_GO: the full re-bin's
// layout is made, its scatter is due; F_TICKET counts the scatter's finished
// workgroups; F_CUR: the store (0 or 1); F_TICK: the tick of the next step,
// modulo 6; F_NITEMS, F_NITEMS1: the containers of either store's layout;
// F_HOLE_LIMIT: more holes than this force a full re-bin at the next step.
enum DevFlag { F_OVERFLOW = 0, F_FORCE = 1, F_GO = 2, F_CUR = 3, F_TICK = 4, F_NITEMS = 5,
               F_NITEMS1 = 6, F_BADINPUT = 7, F_REPACKS = 8, F_LASTMOV = 9, F_TICKET = 10,
               F_STAT_ITEMS = 11, F_STAT_HOLES = 12, F_HOLE_LIMIT = 13, F_COUNT = 16 };

// Counts of holes and of a step's movers, spread over kSpread 64-byte lines
// (hundreds of thousands of workgroups add to them).
constexpr int kSpread = 64;
constexpr int kSpreadInts = kSpread * 16;   // line i: holes at 16 i, movers at 16 i + 1

struct TapeStep {
    const void *u;     // field of the step (borrowed)
    double dt;         // sub-step length
};

constexpr size_t kSavedBytes = (size_t)2 << 30;

struct Block {         // device memory from block_alloc
    void *buf = nullptr;
    size_t bytes = 0;
};
using Snapshot = Block;   // particle store and layout at a checkpoint

// Notes that a launch on s writes the store.
void wrote_store(st_ctx *c, hipStream_t s);
// Whether a read-out on s may use the re-bin's second store (nothing lies in it
// between re-bins): where s wrote the store last, for whoever writes the store or
// reads it from another stream has ordered that stream against s first.  A
// captured read-out may where its capture wrote the store before it, for then
// a replay is ordered as a writer; what is captured changes nothing for calls
// outside.
bool second_store_free(const st_ctx *c, hipStream_t s);

// Device memory of the current device, at least `bytes` of it, perhaps one that
// block_free kept (its contents are anything).
hipError_t block_alloc(int device, size_t bytes, Block *b);
// Takes a block back; nothing on the device may use it any more.
void block_free(int device, Block *b);
// hipMalloc for memory that is not kept; the kept blocks make room for it.
hipError_t device_malloc(void **p, size_t bytes);
// Gives the kept blocks back.
void release_kept();

// One container's run in a saved step or checkpoint.
struct alignas(16) RunItem {
    int32_t c, s0, cnt, k;   // chunk, first slot, slots in use, containers of the chunk
};

// Byte offsets inside a snapshot: the 7 state arrays ([7][slots] of the
// state scalar), ids, the containers' runs with their count, the containers
// themselves and the chunks' first containers.
struct SnapLayout {
    size_t state, id, items, nitems, cont, first, bytes;
};

inline SnapLayout snap_layout(int64_t slots, size_t tsize, int64_t C, int64_t max_items)
{
    auto up64 = [](size_t v) { return (v + 63) & ~(size_t)63; };
    SnapLayout l;
    l.state = 0;
    l.id = 7 * (size_t)slots * tsize;
    l.items = up64(l.id + (size_t)slots * 4);
    l.nitems = l.items + (size_t)max_items * sizeof(RunItem);
    l.cont = up64(l.nitems + 4);
    l.first = l.cont + (size_t)max_items * sizeof(Cont);
    l.bytes = up64(l.first + (size_t)(C + 1) * 4);
    return l;
}

}  // namespace st

struct st_ctx {
    st_mesh_desc desc;
    st::Params prm;
    int device = 0;
    int form = 0;
    size_t tsize = 8;          // bytes of the state scalar
    size_t asize = 8;          // bytes of the source accumulator
    int64_t C = 0;             // chunks
    int64_t cap = 0;           // particle capacity
    int64_t slots = 0;         // slots per store
    int64_t mcap = 0;          // staging capacity of injections
    int64_t nrec = 0;          // records of one tick's inboxes
    st::InboxRule inbox = {0, 0};
    int64_t max_items = 0;     // upper bound of containers
    int64_t count = 0;         // particles in the store (host mirror)
    int64_t pending = 0;       // injected particles waiting in the staging area
    int64_t next_id = 0;
    // stream of the last launch that wrote the store, and, of the last such launch
    // that was captured, stream and capture
    hipStream_t store_stream = nullptr, capture_stream = nullptr;
    unsigned long long capture = 0;

    // device memory
    void *store[2][8] = {};    // SoA arrays of the store and the re-bin's target (F_CUR)
                               // (array k of store b starts past a stagger)
    std::vector<st::Block> blocks;  // allocations that hold the buffers below
    st::Cont *cont[2] = {};    // [max_items] containers of either store
    int32_t *first[2] = {};    // [C+1] first container of each chunk
    void *rec = nullptr;       // [2][nrec] inboxes, by the tick's parity
    void *stage = nullptr;         // [mcap] staged injections
    int32_t *stage_dest = nullptr; // [mcap] their chunks
    int32_t *staged = nullptr;     // [C] their number by chunk, so many apart: a line each,
    int64_t staged_stride = 16;    // since neighbouring chunks are crowded together
    int32_t stage_in_store = 0;    // they are staged in the (empty) store instead
    int32_t *cursor = nullptr;     // [C] scatter cursors of the full re-bin
    int32_t *new_cnt = nullptr;    // [C] particles per chunk at a full re-bin
    int4 *lay = nullptr;           // [C] its layout: first slot, per container, room, containers
    int64_t *lay_sums = nullptr;   // [2] and [C/1024+1]: sums of a layout made in several
    int4 *lay_part = nullptr;      // launches
    int32_t *flags = nullptr;      // DevFlag
    int32_t *spread = nullptr;     // spread counters
    void *src = nullptr;           // [C][3][E^3] accumulator (double or float)
    int32_t *written = nullptr;    // [C] it holds something (else the chunk's is zero)
    st::Block stage64;             // staging for host-side injects ([batch][7] double)

    // tape
    int tape_every = 0;
    std::vector<st::TapeStep> tape;
    std::vector<st::Snapshot> snaps;  // one per tape_every steps
    // kept from a consumed tape for the next one (released by st_tape_clear
    // and st_destroy): checkpoint buffers, and the workspace of st_backward
    // (the state at the end of the forward run, the saved states of one
    // segment, the adjoint records and dL/dS by chunk)
    std::vector<st::Snapshot> spare;
    // the states of the taped steps between checkpoints, by step (no buffer:
    // not kept), and buffers for them from a consumed tape; their bytes in all
    std::vector<st::Block> saved, saved_spare;
    size_t saved_bytes = 0;
    size_t saved_max = st::kSavedBytes;   // less where memory ran out
    st::Block bwd_ws;

    // coupled run
    void *fieldbuf[2] = {};
    hipStream_t side = nullptr;

    // extrapolator-corrector history ([3][ncell] binary64 each), allocated
    // on first use
    double *ec_prev = nullptr;     // S_last of the previous call
    double *ec_ext = nullptr;      // extrapolation made at the previous call

    // step-kernel timing (a pair of events attached to each launch)
    int timing = 0;
    std::vector<hipEvent_t> tev;   // pairs: start, stop

    std::string err;
};

namespace st {

// Kernel launchers (st_device.hip).  All enqueue on `s`.
hipError_t launch_init(st_ctx *c, hipStream_t s);
// places the last step's arrivals (else the next step does)
hipError_t launch_settle(st_ctx *c, hipStream_t s);
// counts the non-empty containers and the holes into F_STAT_*
hipError_t launch_stats(st_ctx *c, hipStream_t s);
// the runs of the (settled) store's containers and their count
hipError_t launch_runs(st_ctx *c, RunItem *items, int32_t *nitems, hipStream_t s);
// takes staged injections from `keep` on out of the counts by chunk again
hipError_t launch_unstage(st_ctx *c, int64_t keep, hipStream_t s);
hipError_t launch_flush_pending(st_ctx *c, hipStream_t s);
hipError_t launch_zero_sources(st_ctx *c, hipStream_t s);
hipError_t launch_zero_i32(int32_t *p, int64_t n, hipStream_t s);
// save (a snapshot buffer, or null): the step also writes there what its
// reverse reads (the state each slot starts with, ids and the layout)
hipError_t launch_step(st_ctx *c, const void *u, double dt, int deposit, hipStream_t s,
                       void *save = nullptr);
hipError_t launch_stage_inject(st_ctx *c, int64_t n, const double *x, const double *up,
                               const double *d, int64_t at, hipStream_t s);
hipError_t launch_get_particles(st_ctx *c, double *x, double *up, double *d, int64_t *id,
                                int32_t *cell, hipStream_t s);
hipError_t launch_get_sources(st_ctx *c, double *out, int reset, hipStream_t s);
hipError_t launch_rotate_field(st_ctx *c, const void *u0, void *out, double cs, double sn,
                               hipStream_t s);
hipError_t launch_snapshot(st_ctx *c, void *dst, int restore, hipStream_t s);
hipError_t launch_ec(st_ctx *c, int kind, const double *S_last, double *applied, hipStream_t s);
hipError_t launch_zero_f64(double *p, int64_t n, hipStream_t s);
size_t snapshot_bytes(const st_ctx *c);
hipError_t launch_backward(st_ctx *c, const double *lam, double *dU, double *dd, hipStream_t s);
// allocates st_backward's workspace for checkpoints every K sub-steps, if smaller
hipError_t reserve_backward(st_ctx *c, int64_t K, bool recompute);
// The states of taped steps take at most kSavedBytes (until st_tape_clear less,
// once memory ran out).  Whether n more fit; a buffer for one more, or none;
// takes the last n steps' back; gives all of them up (their steps are
// recomputed), and whether there were any.
bool saved_fit(const st_ctx *c, int64_t n);
Block take_saved(st_ctx *c);
void untake_saved(st_ctx *c, size_t n);
bool drop_saved(st_ctx *c);
hipError_t launch_hilbert_positions(int32_t order, int64_t nseg, int64_t seg_begin,
                                    int64_t per_seg, const double L[3], int64_t first, int64_t n,
                                    const double *u, double *x, hipStream_t s);
hipError_t launch_bounding_boxes(st_ctx *c, int64_t id0, int64_t per_part, int64_t nparts,
                                 double *box, hipStream_t s);
// The fixed device array of st_bounding_boxes_noalloc (st_hilbert.hip):
// noalloc_scratch_init takes this device's address of it (the device must be
// current; once per device, later calls return at once); noalloc_scratch
// returns that address, or an error if it was never taken.
hipError_t noalloc_scratch_init(int device);
hipError_t launch_stream_copy(const void *src, void *dst, int64_t bytes, hipStream_t s);
hipError_t noalloc_scratch(int device, double **ptr);

template <class T>
Views<T> views_of(const st_ctx *c)
{
    auto v = [&](int b) {
        return View<T>{(T *)c->store[b][0], (T *)c->store[b][1], (T *)c->store[b][2],
                       (T *)c->store[b][3], (T *)c->store[b][4], (T *)c->store[b][5],
                       (T *)c->store[b][6], (int32_t *)c->store[b][7]};
    };
    return Views<T>{v(0), v(1)};
}

// What a kernel that reads the particles gets: both stores, their containers,
// the inboxes and the flags.
template <class T>
struct Store {
    Views<T> V;
    const Cont *cont0, *cont1;
    const MoverRec<T> *rec;   // [2][nrec]
    int64_t nrec;
    const int32_t *flags;
};

template <class T>
Store<T> store_of(const st_ctx *c)
{
    return Store<T>{views_of<T>(c), c->cont[0], c->cont[1], (const MoverRec<T> *)c->rec, c->nrec,
                    c->flags};
}

#ifdef __HIPCC__
// A container's place and its state with index m.
struct ContState {
    int32_t c, base, room, ibase, k, in, cnt, h;
};
__device__ __forceinline__ ContState state_of(const Cont *p, int m)
{
    const Cont d = *p;   // (constant indices: the copy stays in registers)
    return ContState{d.c, d.base, d.room, d.ibase, d.k,
                     m == 0 ? d.in[0] : m == 1 ? d.in[1] : d.in[2],
                     m == 0 ? d.s[0].cnt : m == 1 ? d.s[1].cnt : d.s[2].cnt,
                     m == 0 ? d.s[0].h : m == 1 ? d.s[1].h : d.s[2].h};
}

// The current state of a store: its arrays and containers, and where the
// last step's arrivals are.
template <class T>
struct Current {
    View<T> V;
    const Cont *cont;
    const MoverRec<T> *rec;
    int32_t ni;          // containers
    int32_t m;           // state index of the last step
    __device__ __forceinline__ explicit Current(const Store<T> &s)
    {
        const int cur = s.flags[F_CUR], t = s.flags[F_TICK];
        V = s.V.pick(cur);
        cont = cur ? s.cont1 : s.cont0;
        ni = cur ? s.flags[F_NITEMS1] : s.flags[F_NITEMS];
        m = (t + 2) % 3;
        rec = s.rec + ((t + 1) & 1) * s.nrec;
    }
};
#endif

}  // namespace st
