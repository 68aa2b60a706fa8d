// HIP kernels of the scaletrack library, written for CDNA4 (gfx950, wave64).
//
// One step of the particle method (paper Sec. 2.1 equations of motion and
// momentum source, Sec. 2.5 interpolation, deposit and time integration)
// is three launches:
//   step      one workgroup per container (a run of the slots of one chunk):
//             stage the chunk's fluid tile with a one-cell halo in LDS,
//             gather, integrate, deposit into an LDS accumulator of the
//             chunk's cells, write every particle back in place, collect the
//             chunk crossers ("movers") in LDS by direction and emit them as
//             whole records into the inboxes of the neighbouring chunks'
//             containers, with one atomic instruction for all of a
//             workgroup's reservations, and flush the accumulator with one
//             read-modify-write (or one atomic, for chunks of several
//             containers) per cell.  A mover's slot becomes a hole (binary32:
//             an offset no particle has, written by the step's own store;
//             binary64: its diameter negated, its state left in place).  The
//             container's own arrivals of the step before are taken from its inbox into
//             the holes the stream passes, then past its last slot, where the
//             step's own vector stores write them: no pass of their own, and
//             no scattered writes but their diameters and ids;
//   gate      one workgroup: the next tick; and, when a container ran out of
//             room, an inbox was too small, particles were injected or too
//             many holes gathered, the layout of a full re-bin (counts per
//             chunk, rooms, containers; on meshes of many chunks in three
//             more launches);
//   scatter   only then: a counting sort into the second store, which becomes
//             the store.
#include "st_internal.h"

#include <hip/hip_ext.h>

#include <math.h>

#include <algorithm>

namespace st {
namespace {

__device__ __forceinline__ int64_t wrapi(int64_t i, int64_t n)
{
    int64_t r = i % n;
    return r < 0 ? r + n : r;
}

__device__ __forceinline__ uint64_t lanes_below_mask() { return (1ull << __lane_id()) - 1ull; }

template <class V>
__device__ __forceinline__ V wave_incl_scan(V x)
{
    const int lane = __lane_id();
    for (int o = 1; o < 64; o <<= 1) {
        const V y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    return x;
}

// Block-wide exclusive scan of one value per thread (any multiple of 64
// threads up to 1024); returns the prefix and the block total.
template <class V>
__device__ V block_excl_scan(V v, V &total)
{
    __shared__ V ws[16];
    const int lane = __lane_id(), wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const V incl = wave_incl_scan(v);
    if (lane == 63) ws[wave] = incl;
    __syncthreads();
    if (wave == 0) {
        V w = lane < nw ? ws[lane] : V(0);
        w = wave_incl_scan(w);
        if (lane < nw) ws[lane] = w;
    }
    __syncthreads();
    total = ws[nw - 1];
    const V ex = (wave ? ws[wave - 1] : V(0)) + incl - v;
    __syncthreads();
    return ex;
}

// ---------------------------------------------------------------------------
// chunks and re-basing of chunk-local offsets
// ---------------------------------------------------------------------------
__device__ __forceinline__ int64_t chunk_index(const Params &p, int64_t cx, int64_t cy,
                                               int64_t cz)
{
    return (cz * p.nc[1] + cy) * p.nc[0] + cx;
}

// An offset that left [0, E) moves to the chunk k steps away along the axis
// and is re-based onto it; a rounding that lands exactly on E belongs to the
// next chunk at offset 0.  Returns k.
template <class T>
__device__ __forceinline__ int rebase(T &xi, T fe, T inv_e)
{
    T kf = floor(xi * inv_e);
    int k = (int)kf;
    xi = xi - kf * fe;
    if (xi < T(0)) { xi += fe; --k; }
    if (xi >= fe) { xi -= fe; ++k; }
    return k;
}

template <class T>
__device__ __forceinline__ int64_t chunk_after(const Params &p, int64_t c, T &ox, T &oy, T &oz)
{
    const T fe = T(p.E), inv_e = T(1) / T(p.E);  // E is a power of two: exact
    int kx = rebase(ox, fe, inv_e), ky = rebase(oy, fe, inv_e), kz = rebase(oz, fe, inv_e);
    if ((kx | ky | kz) == 0) return c;
    const int64_t cx = c % p.nc[0];
    const int64_t cy = (c / p.nc[0]) % p.nc[1];
    const int64_t cz = c / ((int64_t)p.nc[0] * p.nc[1]);
    return chunk_index(p, wrapi(cx + kx, p.nc[0]), wrapi(cy + ky, p.nc[1]),
                       wrapi(cz + kz, p.nc[2]));
}

// FP32-everywhere form: the cell of a binary32 coordinate in metres along one
// axis, from the rounded binary32 product x n / L (a rounding that reaches n
// stays in the last cell).  Every kernel takes a particle's cell and chunk
// from this one product, so they agree on them.
__device__ __forceinline__ float gprod(float x, float inv_h) { return __fmul_rn(x, inv_h); }
__device__ __forceinline__ int gcell(float x, float inv_h, int n)
{
    const int c = (int)floorf(gprod(x, inv_h));
    return min(max(c, 0), n - 1);
}

// The chunk of a stored position: chunk-local offsets re-based from chunk c
// (left re-based), or binary32 coordinates in metres (left as they are).
template <class T>
__device__ __forceinline__ int64_t chunk_of_stored(const Params &p, int64_t c, T &x, T &y, T &z)
{
    if (p.global)
        return chunk_index(p, gcell((float)x, p.inv_hf[0], p.n[0]) / p.E,
                           gcell((float)y, p.inv_hf[1], p.n[1]) / p.E,
                           gcell((float)z, p.inv_hf[2], p.n[2]) / p.E);
    return chunk_after(p, c, x, y, z);
}

// ---------------------------------------------------------------------------
// after the step: the next tick, and the layout of a full re-bin
// ---------------------------------------------------------------------------
struct GateArgs {
    Cont *cont0, *cont1;
    int32_t *first0, *first1;
    int32_t *new_cnt, *cursor;
    int4 *lay;
    int32_t *flags, *spread;
    int64_t *sums;           // layout in several launches: particles, weights
    int4 *part;              // and its blocks' sums: slots (64 bits), containers, records
    int64_t C;
    int32_t nc[3];
    int64_t slots;           // slots to share out among the particles and the spare ones
    InboxRule inbox;
    int32_t advance;         // after a step (not for staged injections alone)
    int32_t *staged;         // [C] staged injections to be placed too, or null,
    int64_t stride;          // so many apart
    int32_t one;             // the layout is made by the gate's own workgroup
};

// The layouts of a full re-bin, the present one and the new, and the state
// index after the step.
struct Layouts {
    Cont *ct, *nct;
    const int32_t *cf;
    int32_t *ncf;
    int cur, m;
    __device__ __forceinline__ Layouts(const GateArgs &a, int cur_, int m_) : cur(cur_), m(m_)
    {
        ct = cur ? a.cont1 : a.cont0;
        cf = cur ? a.first1 : a.first0;
        nct = cur ? a.cont0 : a.cont1;
        ncf = cur ? a.first0 : a.first1;
    }
};

// A chunk's particles: those of its containers (their holes out, their inboxes
// and the movers that found them full in), and staged ones.
__device__ __forceinline__ int32_t chunk_total(const GateArgs &a, const Layouts &L, int64_t c)
{
    int32_t n = a.staged ? a.staged[c * a.stride] : 0;
    const int32_t j1 = L.cf[c + 1];
    for (int32_t j = L.cf[c]; j < j1; ++j) {
        const ContState s = state_of(L.ct + j, L.m);
        n += s.cnt - s.h + s.in;
    }
    return n;
}

// Counts them, and sets their places: those that stay in its containers,
// container by container, then its inboxes' records, then (from the cursor
// on) injections and the movers whose inbox was full.
__device__ __forceinline__ int32_t count_chunk(const GateArgs &a, const Layouts &L, int64_t c)
{
    const int32_t j0 = L.cf[c], j1 = L.cf[c + 1];
    int32_t n = 0, all = 0;
    for (int32_t j = j0; j < j1; ++j) {
        L.ct[j].place[0] = n;
        n += L.ct[j].s[L.m].cnt - L.ct[j].s[L.m].h;
    }
    all = n;
    for (int32_t j = j0; j < j1; ++j) {
        L.ct[j].place[1] = n;
        n += min(L.ct[j].in[L.m], inbox_cap(L.ct[j].room, a.inbox));
        all += L.ct[j].in[L.m];
    }
    if (a.staged) all += a.staged[c * a.stride];
    a.new_cnt[c] = all;
    a.cursor[c] = n;
    return all;
}

// Share of the spare slots a chunk asks for in a re-binned layout: the
// largest count among the chunk and its six face neighbours (periodic), plus
// kSlackMin.  What a chunk can gain before the next re-bin is bounded by what
// its neighbours can send, so a sparse chunk at the edge of a dense region
// gets room for the arrivals from the dense side.
template <class F>
__device__ __forceinline__ int64_t room_weight(const F &cnt, const int32_t (&nc)[3], int64_t i)
{
    const int32_t j = (int32_t)i;
    const int32_t sx = 1, sy = nc[0], sz = nc[0] * nc[1];
    const int32_t x = j % nc[0], y = (j / nc[0]) % nc[1], z = j / sz;
    const int32_t nb[6] = {
        j + (x == nc[0] - 1 ? -(nc[0] - 1) * sx : sx), j + (x == 0 ? (nc[0] - 1) * sx : -sx),
        j + (y == nc[1] - 1 ? -(nc[1] - 1) * sy : sy), j + (y == 0 ? (nc[1] - 1) * sy : -sy),
        j + (z == nc[2] - 1 ? -(nc[2] - 1) * sz : sz), j + (z == 0 ? (nc[2] - 1) * sz : -sz)};
    int32_t m = cnt(j);
#pragma unroll
    for (int k = 0; k < 6; ++k) m = max(m, cnt(nb[k]));
    return (int64_t)m + kSlackMin;
}

// A chunk's containers in the new layout: k of at most kSeg particles, equal
// rooms of whole groups of kAlign slots, the spare slots shared out in
// proportion to the chunks' weights and rounded down.
struct Room {
    int32_t n, k, per, room, icap;
};
__device__ __forceinline__ Room chunk_room(const GateArgs &a, int64_t c, int64_t spare,
                                           int64_t denom)
{
    Room r;
    r.n = a.new_cnt[c];
    r.k = r.n > kSeg ? (r.n + kSeg - 1) / kSeg : 1;
    r.per = ((r.n + r.k - 1) / r.k + kAlign - 1) / kAlign * kAlign;
    const int64_t w = room_weight([&](int32_t j) { return a.new_cnt[j]; }, a.nc, c);
    const int64_t extra = spare * w / denom / r.k;
    r.room = (int32_t)min((int64_t)kRoomMax, r.per + extra / kAlign * kAlign);
    r.icap = inbox_cap(r.room, a.inbox);
    return r;
}

__device__ __forceinline__ void write_chunk(const GateArgs &a, const Layouts &L, int64_t c,
                                            const Room &r, int64_t base, int32_t j0, int32_t ib)
{
    L.ncf[c] = j0;
    a.lay[c] = int4{(int32_t)base, r.per, r.room, r.k};
    if (a.staged) a.staged[c * a.stride] = 0;
    for (int32_t i = 0; i < r.k; ++i) {
        Cont d;
        d.c = (int32_t)c;
        d.base = (int32_t)base + i * r.room;
        d.room = r.room;
        d.ibase = ib + i * r.icap;
        d.k = r.k;
        for (int u = 0; u < 3; ++u) {
            d.in[u] = 0;
            d.s[u].cnt = u == L.m ? min(max(r.n - i * r.per, 0), r.per) : 0;
            d.s[u].h = 0;
        }
        d.place[0] = d.place[1] = 0;
        L.nct[j0 + i] = d;
    }
}

__device__ __forceinline__ void finish_layout(const GateArgs &a, const Layouts &L, int32_t ni,
                                              int64_t total)
{
    L.ncf[a.C] = ni;
    a.flags[L.cur ? F_NITEMS : F_NITEMS1] = ni;
    // (of the steps until the next full re-bin: a sixteenth of the particles)
    a.flags[F_HOLE_LIMIT] = (int32_t)(total / 16 + 1024);
}

// One workgroup.  Without a full re-bin (nearly always) it only turns the
// tick and sums the spread counters.  With one, it makes the new layout too, or
// (many chunks) leaves it to the launches below.
__global__ void __launch_bounds__(1024) k_gate(GateArgs a)
{
    int32_t *const f = a.flags;
    const int32_t t = f[F_TICK], cur = f[F_CUR];
    const bool full = (f[F_OVERFLOW] | f[F_FORCE]) != 0;
    int32_t *const l = a.spread + 16 * (threadIdx.x & 63);
    int32_t holes = l[0], movers = l[1];
    __syncthreads();   // every thread has read the flags before one writes them
    if (threadIdx.x < 64) {
        for (int o = 32; o > 0; o >>= 1) {
            holes += __shfl_xor(holes, o);
            movers += __shfl_xor(movers, o);
        }
        l[1] = 0;
        if (full) l[0] = 0;
        if (threadIdx.x == 0) {
            if (a.advance) {
                f[F_LASTMOV] = movers;
                f[F_TICK] = t == 5 ? 0 : t + 1;
            }
            // holes are streamed like particles until a full re-bin drops them
            f[F_FORCE] = !full && holes - movers > f[F_HOLE_LIMIT];
            if (full) {
                f[F_OVERFLOW] = 0;
                f[F_TICKET] = 0;
                f[F_GO] = 1;
                if (!a.one) a.sums[0] = a.sums[1] = 0;
            }
        }
    }
    if (!full || !a.one) return;

    const Layouts L(a, cur, a.advance ? t % 3 : (t + 2) % 3);
    for (int64_t c = threadIdx.x; c < a.C; c += 1024) count_chunk(a, L, c);
    __syncthreads();
    // The particles are counted here, not by the host: a captured step may be
    // replayed after more have been put in.
    int64_t w = 0, np = 0, denom, total;
    for (int64_t c = threadIdx.x; c < a.C; c += 1024) {
        w += room_weight([&](int32_t j) { return a.new_cnt[j]; }, a.nc, c);
        np += a.new_cnt[c];
    }
    block_excl_scan<int64_t>(w, denom);
    block_excl_scan<int64_t>(np, total);
    int64_t slot0 = 0;
    int32_t cont_0 = 0, rec0 = 0;
    for (int64_t r0 = 0; r0 < a.C; r0 += 1024) {
        const int64_t c = r0 + threadIdx.x;
        Room r = {0, 0, 0, 0, 0};
        if (c < a.C) r = chunk_room(a, c, a.slots - total, denom);
        int64_t slots_r;
        int32_t conts_r, recs_r;
        const int64_t base = slot0 + block_excl_scan<int64_t>((int64_t)r.k * r.room, slots_r);
        const int32_t j0 = cont_0 + block_excl_scan<int32_t>(r.k, conts_r);
        const int32_t ib = rec0 + block_excl_scan<int32_t>(r.k * r.icap, recs_r);
        if (c < a.C) write_chunk(a, L, c, r, base, j0, ib);
        slot0 += slots_r;
        cont_0 += conts_r;
        rec0 += recs_r;
    }
    if (threadIdx.x == 0) finish_layout(a, L, cont_0, total);
}

// The same layout over many workgroups, 1024 chunks each, behind the gate: the
// counts and the two sums of them, then each block's slots, containers and
// records, then the layout.  Bound by latency, then by the containers' lines
// (64 B read, 64 B written): 27 + 7 + 14 us at 262144 chunks.
constexpr int kLayBlock = 1024;

__device__ __forceinline__ Layouts gated_layouts(const GateArgs &a)
{
    return Layouts(a, a.flags[F_CUR], (a.flags[F_TICK] + 2) % 3);
}

__global__ void __launch_bounds__(kLayBlock) k_lay_count(GateArgs a)
{
    if (!a.flags[F_GO]) return;
    const Layouts L = gated_layouts(a);
    const int64_t c = (int64_t)blockIdx.x * kLayBlock + threadIdx.x;
    int64_t np = 0, w = 0;
    if (c < a.C) {
        np = count_chunk(a, L, c);
        w = room_weight([&](int32_t j) { return chunk_total(a, L, j); }, a.nc, c);
    }
    int64_t npb, wb;
    block_excl_scan<int64_t>(np, npb);
    block_excl_scan<int64_t>(w, wb);
    if (threadIdx.x == 0) {
        atomicAdd((unsigned long long *)a.sums, (unsigned long long)npb);
        atomicAdd((unsigned long long *)a.sums + 1, (unsigned long long)wb);
    }
}

__device__ __forceinline__ int4 pack_part(int64_t slots, int32_t conts, int32_t recs)
{
    return int4{(int32_t)slots, (int32_t)(slots >> 32), conts, recs};
}
__device__ __forceinline__ int64_t part_slots(const int4 &p)
{
    return (int64_t)(uint32_t)p.x | (int64_t)p.y << 32;
}

__global__ void __launch_bounds__(kLayBlock) k_lay_rooms(GateArgs a)
{
    if (!a.flags[F_GO]) return;
    const int64_t c = (int64_t)blockIdx.x * kLayBlock + threadIdx.x;
    Room r = {0, 0, 0, 0, 0};
    if (c < a.C) r = chunk_room(a, c, a.slots - a.sums[0], a.sums[1]);
    int64_t slots;
    int32_t conts, recs;
    block_excl_scan<int64_t>((int64_t)r.k * r.room, slots);
    block_excl_scan<int32_t>(r.k, conts);
    block_excl_scan<int32_t>(r.k * r.icap, recs);
    if (threadIdx.x == 0) a.part[blockIdx.x] = pack_part(slots, conts, recs);
}

__global__ void __launch_bounds__(kLayBlock) k_lay_write(GateArgs a)
{
    if (!a.flags[F_GO]) return;
    const Layouts L = gated_layouts(a);
    // where the block begins: the blocks before it
    int64_t s = 0, slot0;
    int32_t j = 0, i = 0, cont_0, rec0;
    for (int32_t b = threadIdx.x; b < (int32_t)blockIdx.x; b += kLayBlock) {
        const int4 p = a.part[b];
        s += part_slots(p);
        j += p.z;
        i += p.w;
    }
    block_excl_scan<int64_t>(s, slot0);
    block_excl_scan<int32_t>(j, cont_0);
    block_excl_scan<int32_t>(i, rec0);
    const int64_t c = (int64_t)blockIdx.x * kLayBlock + threadIdx.x;
    Room r = {0, 0, 0, 0, 0};
    if (c < a.C) r = chunk_room(a, c, a.slots - a.sums[0], a.sums[1]);
    int64_t slots_r;
    int32_t conts_r, recs_r;
    const int64_t base = slot0 + block_excl_scan<int64_t>((int64_t)r.k * r.room, slots_r);
    const int32_t j0 = cont_0 + block_excl_scan<int32_t>(r.k, conts_r);
    const int32_t ib = rec0 + block_excl_scan<int32_t>(r.k * r.icap, recs_r);
    if (c < a.C) write_chunk(a, L, c, r, base, j0, ib);
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0)
        finish_layout(a, L, cont_0 + conts_r, a.sums[0]);
}

__global__ void k_set_flag(int32_t *flags, int which, int32_t v) { flags[which] = v; }

// ---------------------------------------------------------------------------
// the step kernel
// ---------------------------------------------------------------------------
template <class T, class A>
struct StepArgs {
    Views<T> V;
    Cont *cont0, *cont1;
    const int32_t *first0, *first1;
    const T *u;              // field [3][n2][n1][n0]
    A *src;                  // [C][3][E^3]
    int32_t *written;        // [C] the chunk's sources hold something (else they are zero)
    MoverRec<T> *rec;        // inboxes [2][nrec]
    int64_t nrec;
    int32_t *flags, *spread;
    InboxRule inbox;
    int32_t deposit;         // 0: move and re-bin only (tape recompute)
    // taped steps and their recomputation: what the reverse of the step reads,
    // saved into a snapshot buffer at the store's slot indices: the state each slot
    // starts the step with, its id, and the containers' runs
    T *sv[7];
    int32_t *sid;
    RunItem *sitems;
    int32_t *snitems;
    Params p;
    T dt;
    T dt_h[3];               // dt / h per axis
    T tau_coef;
    T g[3];
    T g_dt[3];               // g dt
    T mass_coef;             // w rho_p pi / 6
    T inv_V;                 // 1 / cell volume
    T re2_coef;              // (rho_f / mu_f)^2: Re^2 = re2_coef d^2 |u_f - u_p|^2
};

// reciprocal: the hardware's (1 ulp) in binary32, a division in binary64
__device__ __forceinline__ float recip(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double recip(double x) { return 1.0 / x; }

// Re^0.687 from Re^2 (no square root): 2^(0.3435 log2 Re^2) with the
// hardware's base-2 logarithm and exponential in binary32, pow in binary64.
// Re^2 = 0 gives 0 (log2 0 = -inf).
__device__ __forceinline__ float sn_re_pow(float re2)
{
    return __builtin_amdgcn_exp2f(0.3435f * __builtin_amdgcn_logf(re2));
}
__device__ __forceinline__ double sn_re_pow(double re2) { return pow(re2, 0.3435); }

// Workgroups are dispatched round-robin over the 8 XCDs.  Containers are
// dealt to the XCDs in blocks of kXcdBlock consecutive items (neighbouring
// chunks, which share halo cells through the XCD's L2), block j to XCD
// j mod 8, so that every XCD gets a share of every region of their list
// and of its work, however uneven the chunk occupancy.  A bijection of
// [0, R), R their number rounded up to whole rounds of 8 blocks; ids that
// map past them exit.  Blocks of 16 measured best (1.8 % less
// step-kernel time than 64 on 128^3; one container per block, the hardware's own
// dealing, 7 % more).
constexpr int64_t kXcdBlock = 16;
__device__ __forceinline__ int64_t xcd_remap(int64_t bid)
{
    const int64_t x = bid % 8, k = bid / 8;
    return ((k / kXcdBlock) * 8 + x) * kXcdBlock + k % kXcdBlock;
}

// G consecutive values at a G*sizeof(T)-aligned address, as one 16-byte
// access with the non-temporal hint: the particle state is streamed, read
// once and written once per step, so it should not displace what the caches
// hold (the tile, the counters, the inboxes).  Measured: 13 % less step
// kernel time on 1e7 particles, 11 % on 1.4e9.
template <class T, int G>
__device__ __forceinline__ void vld(const T *p, T (&v)[G])
{
    typedef T vec __attribute__((ext_vector_type(G)));
    const vec r =
        __builtin_nontemporal_load((const vec *)__builtin_assume_aligned(p, G * sizeof(T)));
#pragma unroll
    for (int k = 0; k < G; ++k) v[k] = r[k];
}

template <class T, int G>
__device__ __forceinline__ void vst(T *p, const T (&v)[G])
{
    typedef T vec __attribute__((ext_vector_type(G)));
    vec r;
#pragma unroll
    for (int k = 0; k < G; ++k) r[k] = v[k];
    __builtin_nontemporal_store(r, (vec *)__builtin_assume_aligned(p, G * sizeof(T)));
}

// base + byte offset: a uniform 64-bit base plus a 32-bit per-lane offset,
// which the loads and stores take in their scalar-base addressing form
template <class T>
__device__ __forceinline__ T *at_byte(T *base, uint32_t byte_off)
{
    return (T *)((char *)base + byte_off);
}
template <class T>
__device__ __forceinline__ const T *at_byte(const T *base, uint32_t byte_off)
{
    return (const T *)((const char *)base + byte_off);
}

// A slot holds a particle unless its offset is the hole mark (the step kernel
// stores it for a particle that left, in the binary32 forms, and for one whose
// new position is not finite, in all) or its diameter is not positive
// (binary64 form: the diameter of a particle that left is negated).  The
// containers' counts of holes are these slots exactly: arrivals and the places
// of a full re-bin are reckoned from them.
// (A particle whose inbox was full stays in place with the un-rebased, perhaps
// negative, offsets of its new position.)
template <class T>
__device__ __forceinline__ bool occupied(T ox, T d)
{
    return ox > T(kHoleMark) && d > T(0);
}

// Chunk-local offsets outside [0, E) on some axis: those of a mover.  (An
// offset that is not a number is not outside: such a particle, its first
// offset aside, stays in its chunk, where the next step drops it.)
template <class T>
__device__ __forceinline__ bool left_chunk(T x, T y, T z, T fe)
{
    return x < T(0) || x >= fe || y < T(0) || y >= fe || z < T(0) || z >= fe;
}

// Whether no value is NaN or infinite: binary64 by the exponents, binary32 by one
// sum (which may overflow: then this is false too).
template <class T, int G>
__device__ __forceinline__ bool all_finite(const T (&v)[G])
{
    if constexpr (sizeof(T) == 8) {
        uint32_t top = 0;
#pragma unroll
        for (int k = 0; k < G; ++k)
            top = max(top, (uint32_t)__double2hiint(v[k]) & 0x7fffffffu);
        return top < 0x7ff00000u;
    } else {
        T sum = v[0];
#pragma unroll
        for (int k = 1; k < G; ++k) sum += v[k];
        return fabs(sum) < T(INFINITY);
    }
}

// Where a container takes arrivals of the step with state index m (the state
// before it: index pm): slots free for them whatever the step's departures
// (more force the full re-bin), the records its inbox holds, and its first.
struct Inbox {
    int32_t free, cap, base;
};
__device__ __forceinline__ Inbox inbox_of(const Cont *d, int pm, InboxRule rule)
{
    const int32_t room = d->room;
    return Inbox{room - (d->s[pm].cnt - d->s[pm].h) - d->in[pm], inbox_cap(room, rule), d->ibase};
}

// The container of chunk c that container `item` sends its movers to.
__device__ __forceinline__ int32_t container_for(const int32_t *first, int64_t c, int32_t item)
{
    const int32_t f = first[c], k = first[c + 1] - f;
    return f + (k > 1 ? item % k : 0);
}

// A mover sent by itself (farther than one chunk, or more movers than the LDS
// stage holds): x, y, z its new position as stored (un-rebased offsets,
// relative to chunk c).  Returns false when the inbox is full: the particle
// then stays in place (the full re-bin that this forces takes it from there).
template <class T, class A>
__device__ __forceinline__ bool send_mover(const StepArgs<T, A> &a, Cont *ct,
                                           const int32_t *first, MoverRec<T> *rec, int m, int pm,
                                           int32_t item, int64_t c, T x, T y, T z, T vx, T vy,
                                           T vz, T dd, int32_t id)
{
    const int64_t cn = chunk_of_stored(a.p, c, x, y, z);
    const int32_t j = container_for(first, cn, item);
    const Inbox in = inbox_of(ct + j, pm, a.inbox);
    const int32_t r = atomicAdd(&ct[j].in[m], 1);
    if (r >= in.free) a.flags[F_OVERFLOW] = 1;
    if (r >= in.cap) {
        a.flags[F_OVERFLOW] = 1;
        return false;
    }
    rec[in.base + r] = MoverRec<T>{x, y, z, vx, vy, vz, dd, id};
    return true;
}

// Staged mover: its slot within the container (below kRoomMax, 15 bits), its
// direction class (0..26 the neighbouring chunks, 27 farther; 5 bits) and its
// rank within that class (below kMoverStage, 9 bits).
constexpr int kSlotBits = 15, kDirBits = 5;
static_assert(kRoomMax <= (1 << kSlotBits) && kMoverStage <= (1 << (32 - 1 - kSlotBits - kDirBits)),
              "staged mover fields must fit one int32");
static_assert(kDirBits * 4 <= 32, "direction classes of a group must fit one uint32");

// Bound by HBM where the chunks are full: 13 streams of 16-byte accesses and
// the records reach 4.5-4.9 TB/s of the 6.2 that a copy does (1e7 droplets on
// 128^3: 138 us); by the chain of tile, flush and records where they are sparse
// (1500 droplets a container, 4e8 on 512^3: 7.8 ms for 31 GB); and by that chain
// alone on meshes that leave CUs idle.  The arrivals ride in the stream that the
// container writes anyway: a pass of their own, eight scattered 4-byte writes
// each, and the counts it needed took 10 + 7 of 153 us a step at 1e7 (148 now),
// 4.9 + 4.7 of 53 at 777777 (33 now, the LDS sums in binary64 included) and 1.2
// of 8.7 ms at 4e8.  Four workgroups share a CU in binary32 (40 KB of LDS, at
// most 124 VGPRs); five without the prefetched group (32 KB, 95 VGPRs) were
// slower (167 against 158 us a step with its sources), and fewer, larger
// workgroups too, but for small meshes (launch_step_t).
template <class T, class A, int E, int INTERP, int DRAG, bool SAVE, int NB>
__global__ void __launch_bounds__(NB)
     k_step(StepArgs<T, A> a)
{
    constexpr int S = E + 2;            // tile edge with the halo
    constexpr int S3 = S * S * S;
    constexpr int E3 = E * E * E;
    constexpr int G = 16 / sizeof(T);   // consecutive particles per thread
    constexpr int MS = NB < 256 ? kMoverStage / 3 : kMoverStage;   // movers staged
    constexpr int KP = NB < kPool ? NB : kPool;                    // arrivals staged
    static_assert(kAlign % G == 0, "chunk rooms must hold whole particle groups");
    __shared__ T tile[3 * S3];
    // (binary64 in every form: LDS adds of binary32 values take twice as long on
    // this chip; 777777 droplets with Schiller-Naumann drag in the FP32-everywhere
    // form: 47 against 55 us)
    __shared__ double acc[3 * E3];
    __shared__ int32_t mstage[MS];
    // binary32 state: the staged movers' new positions and velocities (9 KB,
    // which with the arrivals still lets four workgroups share a CU; the
    // binary64 form re-reads them instead)
    constexpr bool kStageVals = sizeof(T) == 4;
    __shared__ T mval[kStageVals ? 6 * MS : 1];
    __shared__ MoverRec<T> pool[KP];   // the first arrivals
    __shared__ int32_t mcount, apop, nlost;
    __shared__ int32_t dcount[28], dbase[27];
    __shared__ int32_t nbj[27];           // the neighbouring chunks' containers
    __shared__ Inbox nbin[27];

    // the grid covers the most containers a layout can have, rounded up to
    // whole rounds of the remap
    const int64_t item = xcd_remap(blockIdx.x);
    const int32_t cur = a.flags[F_CUR], tick = a.flags[F_TICK];
    const int32_t ni = cur ? a.flags[F_NITEMS1] : a.flags[F_NITEMS];
    if constexpr (SAVE)
        if (blockIdx.x == 0 && threadIdx.x == 0) *a.snitems = ni;
    if (item >= ni) return;
    Cont *const ct = cur ? a.cont1 : a.cont0;
    const int32_t *const first = cur ? a.first1 : a.first0;
    const View<T> V = a.V.pick(cur);
    // state indices of this step, the one before and the one after
    const int m = tick >= 3 ? tick - 3 : tick, pm = m == 0 ? 2 : m - 1, qm = m == 2 ? 0 : m + 1;
    MoverRec<T> *const rec_in = a.rec + (tick & 1 ? 0 : a.nrec);    // written by the last step
    MoverRec<T> *const rec_out = a.rec + (tick & 1 ? a.nrec : 0);
    const ContState me = state_of(ct + item, pm);
    const int64_t c = me.c;
    const int64_t s0 = me.base;
    const int32_t n_in = me.in, nq_old = me.cnt, h_old = me.h;
    // the arrivals take the holes, then slots past the last
    const int nq = nq_old + max(0, n_in - h_old);
    const int32_t h_left = max(0, h_old - n_in);
    const bool multi = me.k > 1;
    if constexpr (SAVE)
        if (threadIdx.x == 0) a.sitems[item] = RunItem{me.c, me.base, nq, me.k};
    if (threadIdx.x == 0 && ct[item].in[qm] != 0) ct[item].in[qm] = 0;
    if (nq == 0) {   // (mostly as it has been: its line stays clean)
        if (threadIdx.x == 0 && (ct[item].s[m].cnt | ct[item].s[m].h) != 0)
            ct[item].s[m] = {0, 0};
        return;
    }
    const Params &p = a.p;
    const int row = me.c / p.nc[0], cx = me.c - row * p.nc[0];
    const int cz = row / p.nc[1], cy = row - cz * p.nc[1];
    const int64_t ncell = (int64_t)p.n[0] * p.n[1] * p.n[2];

    // A chunk of one container stores its sums over sources that the last
    // read-out cleared (it only marks them) and adds to others.
    const bool add = a.deposit && (multi || a.written[c] != 0);

    // The container's slots are read in groups of G consecutive slots through
    // uniform base pointers and 32-bit offsets (below kRoomMax).  s0 is a
    // multiple of G, and a group that runs past the last slot stays inside the
    // container's room.
    const int ngroups = (nq + G - 1) / G;
    T *const pox = V.ox + s0, *const poy = V.oy + s0, *const poz = V.oz + s0;
    T *const pvx = V.vx + s0, *const pvy = V.vy + s0, *const pvz = V.vz + s0;
    T *const pd = V.d + s0;
    int32_t *const pid = V.id + s0;
    auto load_group = [&](int gi, T (&X)[G], T (&Y)[G], T (&Z)[G], T (&UX)[G], T (&UY)[G],
                          T (&UZ)[G], T (&DD)[G]) {
        const uint32_t ob = (uint32_t)gi * G * (uint32_t)sizeof(T);
        vld<T, G>(at_byte((const T *)pox, ob), X);
        vld<T, G>(at_byte((const T *)poy, ob), Y);
        vld<T, G>(at_byte((const T *)poz, ob), Z);
        vld<T, G>(at_byte((const T *)pvx, ob), UX);
        vld<T, G>(at_byte((const T *)pvy, ob), UY);
        vld<T, G>(at_byte((const T *)pvz, ob), UZ);
        vld<T, G>(at_byte((const T *)pd, ob), DD);
    };

    // Stage the fluid tile: cells E*c - 1 .. E*c + E per axis, wrapped.  The
    // main loop is software-pipelined: a group's loads are issued before the
    // arithmetic of the previous one, and the first group's right after the
    // tile's loads, so that memory latency overlaps work.
    constexpr int NT = (3 * S3 + NB - 1) / NB;
    T vals[NT];
    {
        const int ox0 = cx * E - 1, oy0 = cy * E - 1, oz0 = cz * E - 1;
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            const int t = threadIdx.x + u * NB;
            if (t < 3 * S3) {
                const int comp = t / S3;
                const int r = t - comp * S3;
                const int k = r / (S * S);
                const int j = (r / S) % S;
                const int i = r % S;
                int gx = ox0 + i, gy = oy0 + j, gz = oz0 + k;
                gx += gx < 0 ? p.n[0] : 0;
                gx -= gx >= p.n[0] ? p.n[0] : 0;
                gy += gy < 0 ? p.n[1] : 0;
                gy -= gy >= p.n[1] ? p.n[1] : 0;
                gz += gz < 0 ? p.n[2] : 0;
                gz -= gz >= p.n[2] ? p.n[2] : 0;
                vals[u] = a.u[comp * ncell + ((int64_t)gz * p.n[1] + gy) * p.n[0] + gx];
            }
        }
    }
    // the container's first arrivals, in 16-byte pieces
    constexpr int RV = sizeof(MoverRec<T>) / 16;
    int4 arr[RV];
    const bool have_arr = (int)threadIdx.x < min(n_in, KP);
#pragma unroll
    for (int u = 0; u < RV; ++u)
        arr[u] = have_arr ? reinterpret_cast<const int4 *>(rec_in + me.ibase + threadIdx.x)[u]
                          : int4{0, 0, 0, 0};
    int gi = threadIdx.x;
    T X[G], Y[G], Z[G], UX[G], UY[G], UZ[G], DD[G];
    if (gi < ngroups) load_group(gi, X, Y, Z, UX, UY, UZ, DD);
    // The neighbouring chunks' inboxes, a lane each, needed after the loop: read
    // ahead of it for 8^3-cell chunks, which nearly always have movers, and for
    // smaller ones only when there are some (27 lines a container: 3 to 10 % of a
    // step of 1 to 60 droplets a chunk).
    constexpr bool kEarly = E == 8;
    int32_t nb = 0;
    Inbox nb_in = {0, 0, 0};
    auto neighbour = [&]() {
        const int l = threadIdx.x;
        auto wrap1 = [](int i, int n) { return i < 0 ? i + n : i >= n ? i - n : i; };
        const int64_t dc = chunk_index(p, wrap1(cx + l % 3 - 1, p.nc[0]),
                                       wrap1(cy + (l / 3) % 3 - 1, p.nc[1]),
                                       wrap1(cz + l / 9 - 1, p.nc[2]));
        nb = ni == (int32_t)p.C ? (int32_t)dc : container_for(first, dc, (int32_t)item);
        nb_in = inbox_of(ct + nb, pm, a.inbox);
    };
    if (kEarly && threadIdx.x < 27) neighbour();
#pragma unroll
    for (int u = 0; u < NT; ++u) {
        const int t = threadIdx.x + u * NB;
        if (t < 3 * S3) tile[t] = vals[u];
    }
    for (int t = threadIdx.x; t < 3 * E3; t += NB) acc[t] = 0.0;
    if (threadIdx.x < 28) dcount[threadIdx.x] = 0;
    if (have_arr) {
#pragma unroll
        for (int u = 0; u < RV; ++u) reinterpret_cast<int4 *>(pool + threadIdx.x)[u] = arr[u];
    }
    if (threadIdx.x == 0) mcount = apop = nlost = 0;
    __syncthreads();
    bool pool_open = n_in > 0;   // of the wave: arrivals may be left

    const T dt = a.dt;
    const T fe = T(E), inv_e = T(1) / T(E);
    // FP32-everywhere form: positions in binary32 metres, the cell arithmetic
    // in binary32 (the chunk origin in cells is exact)
    constexpr bool GLOBAL = sizeof(A) == 4;
    const T org[3] = {T(cx * E), T(cy * E), T(cz * E)};
    for (; gi < ngroups; gi += NB) {
        T Xn[G], Yn[G], Zn[G], UXn[G], UYn[G], UZn[G], DDn[G];
        if (gi + NB < ngroups) load_group(gi + NB, Xn, Yn, Zn, UXn, UYn, UZn, DDn);
        const uint32_t o = (uint32_t)gi * G;
        const uint32_t ob = o * (uint32_t)sizeof(T);
        int32_t I[G];
        if constexpr (SAVE) vld<int32_t, G>(at_byte((const int32_t *)pid, o * 4u), I);
        if (pool_open) {
            // holes of the run, and its slots past the last step's last, take
            // arrivals while there are any: one LDS reservation per wave, the
            // lanes' shares from a ballot per bit of their counts (at most 4)
            uint32_t holes = 0;
#pragma unroll
            for (int k = 0; k < G; ++k) {
                const int q = (int)o + k;
                if (q < nq && (q >= nq_old || !occupied(X[k], DD[k]))) holes |= 1u << k;
            }
            if (__ballot(holes != 0)) {
                const int mine = __popc(holes);
                const uint64_t below = lanes_below_mask();
                int ex = 0, tot = 0;
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    const uint64_t bal = __ballot((mine >> b) & 1);
                    ex += __popcll(bal & below) << b;
                    tot += __popcll(bal) << b;
                }
                const int lead = __ffsll((long long)__ballot(1)) - 1;
                int r0 = 0;
                if (__lane_id() == lead) r0 = atomicAdd(&apop, tot);
                r0 = __shfl(r0, lead);
                pool_open = r0 + tot < n_in;
                int r = r0 + ex;
#pragma unroll
                for (int k = 0; k < G; ++k) {
                    if (!((holes >> k) & 1)) continue;
                    if (r < n_in) {
                        auto take = [&](const MoverRec<T> &rc) {
                            X[k] = rc.ox;
                            Y[k] = rc.oy;
                            Z[k] = rc.oz;
                            UX[k] = rc.vx;
                            UY[k] = rc.vy;
                            UZ[k] = rc.vz;
                            DD[k] = rc.d;
                            if constexpr (SAVE) I[k] = rc.id;
                            pd[o + k] = rc.d;
                            pid[o + k] = rc.id;
                        };
                        if (r < KP) take(pool[r]);
                        else take(rec_in[me.ibase + r]);
                    }
                    ++r;
                }
            }
        }
        if constexpr (SAVE) {   // the group as the step finds it, with its ids
            vst<T, G>(at_byte(a.sv[0] + s0, ob), X);
            vst<T, G>(at_byte(a.sv[1] + s0, ob), Y);
            vst<T, G>(at_byte(a.sv[2] + s0, ob), Z);
            vst<T, G>(at_byte(a.sv[3] + s0, ob), UX);
            vst<T, G>(at_byte(a.sv[4] + s0, ob), UY);
            vst<T, G>(at_byte(a.sv[5] + s0, ob), UZ);
            vst<T, G>(at_byte(a.sv[6] + s0, ob), DD);
            vst<int32_t, G>(at_byte(a.sid + s0, o * 4u), I);
        }
        uint32_t movers = 0, dirs = 0;   // mover bits and 5-bit direction classes
#pragma unroll
        for (int k = 0; k < G; ++k) {
            // slots past the run and holes hold no particle
            const bool valid = (int)o + k < nq && occupied(X[k], DD[k]);
            T xi[3] = {X[k], Y[k], Z[k]};   // cell units from the chunk origin
            if constexpr (GLOBAL) {
                xi[0] = gprod(X[k], p.inv_hf[0]) - org[0];
                xi[1] = gprod(Y[k], p.inv_hf[1]) - org[1];
                xi[2] = gprod(Z[k], p.inv_hf[2]) - org[2];
            }
            const T up[3] = {UX[k], UY[k], UZ[k]};
            const T dp = DD[k];

            // gather the fluid velocity at the particle
            T uf[3];
            int cl[3];
            if (INTERP == 0) {
                T f[3];
                int i0[3];
                for (int ax = 0; ax < 3; ++ax) {
                    const T s = xi[ax] - T(0.5);
                    const T fl = floor(s);
                    // -1 .. E-1 for offsets in [0, E); clamped so that no
                    // state can index outside the tile
                    i0[ax] = min(max((int)fl, -1), E - 1);
                    f[ax] = s - fl;
                    cl[ax] = min(max((int)xi[ax], 0), E - 1);
                }
                const int t0 = ((i0[2] + 1) * S + (i0[1] + 1)) * S + (i0[0] + 1);
                const T wx0 = T(1) - f[0], wx1 = f[0];
                const T wy0 = T(1) - f[1], wy1 = f[1];
                const T wz0 = T(1) - f[2], wz1 = f[2];
                const T w00 = wy0 * wz0, w10 = wy1 * wz0, w01 = wy0 * wz1, w11 = wy1 * wz1;
                for (int comp = 0; comp < 3; ++comp) {
                    const T *tc = tile + comp * S3 + t0;
                    const T r00 = wx0 * tc[0] + wx1 * tc[1];
                    const T r10 = wx0 * tc[S] + wx1 * tc[S + 1];
                    const T r01 = wx0 * tc[S * S] + wx1 * tc[S * S + 1];
                    const T r11 = wx0 * tc[S * S + S] + wx1 * tc[S * S + S + 1];
                    uf[comp] = w00 * r00 + w10 * r10 + w01 * r01 + w11 * r11;
                }
            } else {
                for (int ax = 0; ax < 3; ++ax) cl[ax] = min(max((int)xi[ax], 0), E - 1);
                const int t0 = ((cl[2] + 1) * S + (cl[1] + 1)) * S + (cl[0] + 1);
                for (int comp = 0; comp < 3; ++comp) uf[comp] = tile[comp * S3 + t0];
            }

            // semi-implicit Euler, drag implicit and gravity explicit:
            //   u_p' = (tau u_p + dt u_f + tau dt g) / (tau + dt)
            // written as the velocity change, which keeps its relative
            // accuracy in binary32:  u_p' - u_p = dt (u_f - u_p + tau g) / (tau + dt)
            T tau = a.tau_coef * dp * dp;
            if (DRAG == 1) {
                // Schiller-Naumann: tau / (1 + 0.15 Re^0.687), Re from the
                // slip at the start of the step
                const T sx = uf[0] - up[0], sy = uf[1] - up[1], sz = uf[2] - up[2];
                const T re2 = a.re2_coef * (dp * dp) * (sx * sx + sy * sy + sz * sz);
                tau = tau * recip(T(1) + T(0.15) * sn_re_pow(re2));
            }
            const T rD = dt * recip(tau + dt);
            T upn[3], xn[3];
            for (int ax = 0; ax < 3; ++ax) {
                upn[ax] = up[ax] + rD * ((uf[ax] - up[ax]) + tau * a.g[ax]);
                xn[ax] = xi[ax] + upn[ax] * a.dt_h[ax];
            }

            // drag impulse J = m (u_p' - u_p - g dt) = m dt (u_f - u_p - g dt) / (tau + dt),
            // evaluated from the stored inputs (not from the rounded new
            // velocity) and summed in the accumulator precision; the fluid
            // receives -J / V in the start-of-step cell
            if (a.deposit && valid) {
                const T coef = -(a.mass_coef * dp * dp * dp) * rD * a.inv_V;
                const int cell = (cl[2] * E + cl[1]) * E + cl[0];
                for (int ax = 0; ax < 3; ++ax) {
                    const T slip = (uf[ax] - up[ax]) - a.g_dt[ax];
                    atomicAdd(&acc[ax * E3 + cell], (double)(coef * slip));
                }
            }

            // relocate: a particle whose new offset left [0, E) on some axis
            // (left_chunk) crossed into another chunk; it keeps the un-rebased offsets
            // (relative to this chunk) until it is emitted and re-based.  A
            // particle that stays needs no re-basing.  FP32-everywhere form:
            // the new position in metres, wrapped, and its chunk from its cells
            bool mover;
            int gk[3] = {0, 0, 0};   // FP32-everywhere: chunk steps per axis
            if constexpr (GLOBAL) {
                const T xg[3] = {X[k], Y[k], Z[k]};
                for (int ax = 0; ax < 3; ++ax) {
                    T v = xg[ax] + upn[ax] * dt;
                    if (v >= p.Lf[ax]) v -= p.Lf[ax];
                    else if (v < T(0)) v += p.Lf[ax];
                    if (!(v >= T(0) && v < p.Lf[ax])) {   // moved more than a domain length
                        v = fmodf(v, p.Lf[ax]);
                        if (v < T(0)) v += p.Lf[ax];
                    }
                    if (v >= p.Lf[ax]) v = T(0);
                    xn[ax] = v;
                    const int cc = ax == 0 ? cx : ax == 1 ? cy : cz;
                    int dk = gcell(v, p.inv_hf[ax], p.n[ax]) / E - cc;
                    // the shorter way round the periodic domain
                    if (dk > 1 && dk == p.nc[ax] - 1) dk = -1;
                    if (dk < -1 && dk == 1 - p.nc[ax]) dk = 1;
                    gk[ax] = dk;
                }
                mover = (gk[0] | gk[1] | gk[2]) != 0;
            } else {
                // (written out: through left_chunk the binary64 kernel takes 30
                // registers more, one wave a SIMD less)
                mover = xn[0] < T(0) || xn[0] >= fe || xn[1] < T(0) || xn[1] >= fe ||
                        xn[2] < T(0) || xn[2] >= fe;
            }
            if (valid) {   // a hole keeps what it holds (binary32: its mark)
                X[k] = xn[0];
                Y[k] = xn[1];
                Z[k] = xn[2];
                UX[k] = upn[0];
                UY[k] = upn[1];
                UZ[k] = upn[2];
            }
            if (valid && mover) {
                movers |= 1u << k;
                // (a hole's mark in place would not be told from such an offset)
                if (xn[0] <= T(kHoleMark)) X[k] = -T(INFINITY);
                int kx = gk[0], ky = gk[1], kz = gk[2];
                if constexpr (!GLOBAL) {
                    T tx = xn[0], ty = xn[1], tz = xn[2];
                    kx = rebase(tx, fe, inv_e);
                    ky = rebase(ty, fe, inv_e);
                    kz = rebase(tz, fe, inv_e);
                }
                auto near = [](int v) { return (uint32_t)v + 1u <= 2u; };
                const int dir = near(kx) && near(ky) && near(kz)
                                    ? (kx + 1) + 3 * (ky + 1) + 9 * (kz + 1) : 27;
                dirs |= (uint32_t)dir << (kDirBits * k);
            }
        }
        // A first offset that is not finite (from a field or a velocity that is
        // not): the droplet has no place any more, and its slot is a hole like
        // any other (a hole's own offset is finite).  It costs 1 % of the binary64
        // step with Schiller-Naumann drag (1e7 on 128^3: 320 -> 325 us; a binary64
        // sum or a test per droplet 327), and nothing that can be measured elsewhere.
        if (!all_finite(X)) {
#pragma unroll
            for (int k = 0; k < G; ++k)
                if ((int)o + k < nq && DD[k] > T(0) && !(fabs(X[k]) < T(INFINITY))) {
                    movers &= ~(1u << k);
                    X[k] = T(2 * kHoleMark);
                    atomicAdd(&nlost, 1);
                }
        }
        // stage the movers with their direction class: one reservation of
        // stage entries per wave (their ranks within the direction classes
        // are taken after the loop)
        if (__ballot(movers != 0)) {
            // prefix of the lanes' mover counts (at most G < 8) from one
            // ballot per bit; the first active lane reserves for the wave
            const int mine = __popc(movers);
            const uint64_t below = lanes_below_mask();
            int ex = 0, tot = 0;
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const uint64_t bal = __ballot((mine >> b) & 1);
                ex += __popcll(bal & below) << b;
                tot += __popcll(bal) << b;
            }
            const int lead = __ffsll((long long)__ballot(1)) - 1;
            int j0 = 0;
            if (__lane_id() == lead) j0 = atomicAdd(&mcount, tot);
            int j = __shfl(j0, lead) + ex;
            if constexpr (kStageVals) {
                // binary32: the new state too, so that it need not be re-read
#pragma unroll
                for (int k = 0; k < G; ++k) {
                    if (!((movers >> k) & 1)) continue;
                    if (j < MS) {
                        const int dir = (dirs >> (kDirBits * k)) & ((1 << kDirBits) - 1);
                        mstage[j] = (int32_t)(o + k) | (dir << kSlotBits);
                        mval[j] = X[k];
                        mval[MS + j] = Y[k];
                        mval[2 * MS + j] = Z[k];
                        mval[3 * MS + j] = UX[k];
                        mval[4 * MS + j] = UY[k];
                        mval[5 * MS + j] = UZ[k];
                        X[k] = T(2 * kHoleMark);   // the slot becomes a hole
                    } else {  // more movers than the LDS stage holds
                        if (send_mover(a, ct, first, rec_out, m, pm, (int32_t)item, c, X[k], Y[k],
                                       Z[k], UX[k], UY[k], UZ[k], DD[k], pid[o + k]))
                            X[k] = T(2 * kHoleMark);
                    }
                    ++j;
                }
            } else {
                while (movers) {
                    const int k = __ffs(movers) - 1;
                    movers &= movers - 1;
                    if (j < MS) {
                        const int dir = (dirs >> (kDirBits * k)) & ((1 << kDirBits) - 1);
                        mstage[j] = (int32_t)(o + k) | (dir << kSlotBits);
                    } else {  // more movers than the LDS stage holds
                        // binary64: the negated diameter marks the hole
                        if (send_mover(a, ct, first, rec_out, m, pm, (int32_t)item, c, X[k], Y[k],
                                       Z[k], UX[k], UY[k], UZ[k], DD[k], pid[o + k]))
                            pd[o + k] = -DD[k];
                    }
                    ++j;
                }
            }
        }
        // slots past the run in the last group are dead; writing them is harmless
        vst<T, G>(at_byte(pox, ob), X);
        vst<T, G>(at_byte(poy, ob), Y);
        vst<T, G>(at_byte(poz, ob), Z);
        vst<T, G>(at_byte(pvx, ob), UX);
        vst<T, G>(at_byte(pvy, ob), UY);
        vst<T, G>(at_byte(pvz, ob), UZ);
#pragma unroll
        for (int k = 0; k < G; ++k) {
            X[k] = Xn[k];
            Y[k] = Yn[k];
            Z[k] = Zn[k];
            UX[k] = UXn[k];
            UY[k] = UYn[k];
            UZ[k] = UZn[k];
            DD[k] = DDn[k];
        }
    }
    // The chunk's source cells are read while the other waves finish (a chunk
    // of one container adds its sums to them; one of several adds atomically,
    // onto sources that are never left merely marked as cleared).
    A *const src_c = a.src + c * (3 * E3);
    constexpr int NF = (3 * E3 + NB - 1) / NB;
    A old[NF];
    const bool rmw = a.deposit && !multi;
    if (rmw) {
#pragma unroll
        for (int u = 0; u < NF; ++u) {
            const int t = threadIdx.x + u * NB;
            old[u] = add && t < 3 * E3 ? src_c[t] : A(0);
        }
    }
    if (kEarly && threadIdx.x < 27) {
        nbj[threadIdx.x] = nb;
        nbin[threadIdx.x] = nb_in;
    }
    __syncthreads();
    if (!kEarly && threadIdx.x < 27 && mcount > 0) {
        neighbour();
        nbj[threadIdx.x] = nb;
        nbin[threadIdx.x] = nb_in;
    }

    // Mover reservations, all issued by one wave at once: one reservation per
    // neighbouring destination instead of one per mover, which would serialise
    // on the counters of crowded chunks, and the workgroup's share of the
    // spread counters.  The movers' state is read in the same round trip.
    const int nm = min(mcount, MS);
    // ranks of the staged movers within their direction classes
    if (nm > 0) {
        for (int j = threadIdx.x; j < nm; j += NB) {
            const int32_t w = mstage[j];
            const int dir = (w >> kSlotBits) & ((1 << kDirBits) - 1);
            mstage[j] = w | (atomicAdd(&dcount[dir], 1) << (kSlotBits + kDirBits));
        }
        __syncthreads();
    }
    constexpr int NM = (MS + NB - 1) / NB;   // staged movers per thread
    T mx[NM], my[NM], mz[NM], mvx[NM], mvy[NM], mvz[NM], md[NM];
    int32_t mid[NM];
#pragma unroll
    for (int u = 0; u < NM; ++u) {
        const int j = threadIdx.x + u * NB;
        if (j < nm) {
            const int64_t q = s0 + (mstage[j] & ((1 << kSlotBits) - 1));
            if constexpr (kStageVals) {
                mx[u] = mval[j];
                my[u] = mval[MS + j];
                mz[u] = mval[2 * MS + j];
                mvx[u] = mval[3 * MS + j];
                mvy[u] = mval[4 * MS + j];
                mvz[u] = mval[5 * MS + j];
            } else {
                mx[u] = V.ox[q];
                my[u] = V.oy[q];
                mz[u] = V.oz[q];
                mvx[u] = V.vx[q];
                mvy[u] = V.vy[q];
                mvz[u] = V.vz[q];
            }
            md[u] = V.d[q];
            mid[u] = V.id[q];
        }
    }
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        const int n = lane < 27 ? dcount[lane] : 0;
        const int32_t h_new = h_left + mcount + nlost;
        if (lane == 0) ct[item].s[m] = {nq, h_new};
        // one atomic instruction (the counters differ per lane, but for those
        // of a mesh of one or two chunks along an axis)
        int32_t *ctr = nullptr;
        int add = n;
        if (n > 0) ctr = &ct[nbj[lane]].in[m];
        int32_t *const line = a.spread + 16 * (blockIdx.x % kSpread);
        if (lane == 32) {
            ctr = line;
            add = h_new - h_old;
        }
        if (lane == 33) {
            ctr = line + 1;
            add = mcount;
        }
        if (add != 0) {
            const int32_t r = atomicAdd(ctr, add);
            if (n > 0) {
                dbase[lane] = r;
                // arrivals must fit the destination's free slots, else the
                // full re-bin runs
                if (r + n > nbin[lane].free) a.flags[F_OVERFLOW] = 1;
            }
        }
    }

    // flush the chunk's accumulated source
    if (rmw) {
#pragma unroll
        for (int u = 0; u < NF; ++u) {
            const int t = threadIdx.x + u * NB;
            if (t < 3 * E3) src_c[t] = (A)(old[u] + acc[t]);
        }
        if (!add && threadIdx.x == 0) a.written[c] = 1;
    } else if (a.deposit) {
        for (int t = threadIdx.x; t < 3 * E3; t += NB) {
            const A v = (A)acc[t];
            if (v != A(0)) atomicAdd(src_c + t, v);
        }
    }
    if (nm == 0) return;
    __syncthreads();

    // emit the staged movers into their destinations' inboxes
#pragma unroll
    for (int u = 0; u < NM; ++u) {
        const int j = threadIdx.x + u * NB;
        if (j >= nm) continue;
        const int32_t w = mstage[j];
        const int32_t off = w & ((1 << kSlotBits) - 1);
        const int dir = (w >> kSlotBits) & ((1 << kDirBits) - 1);
        const int rank = w >> (kSlotBits + kDirBits);
        bool sent;
        if (dir < 27) {   // within the direction's reservation
            // re-base the offsets into the destination chunk (FP32-everywhere
            // form: positions in metres stay as they are)
            T rx = mx[u], ry = my[u], rz = mz[u];
            chunk_of_stored(p, c, rx, ry, rz);
            const int32_t r = dbase[dir] + rank;
            sent = r < nbin[dir].cap;
            if (sent)
                rec_out[nbin[dir].base + r] =
                    MoverRec<T>{rx, ry, rz, mvx[u], mvy[u], mvz[u], md[u], mid[u]};
            else
                a.flags[F_OVERFLOW] = 1;
        } else {          // farther than one chunk: a reservation of its own
            sent = send_mover(a, ct, first, rec_out, m, pm, (int32_t)item, c, mx[u], my[u], mz[u],
                              mvx[u], mvy[u], mvz[u], md[u], mid[u]);
        }
        // the slot becomes a hole (binary32: the step stored its mark;
        // binary64: the diameter is negated); a particle whose inbox is full
        // stays in place (its un-rebased offsets) for the full re-bin
        if constexpr (kStageVals) {
            if (!sent) pox[off] = mx[u];
        } else {
            if (sent) pd[off] = -md[u];
        }
    }
}


// ---------------------------------------------------------------------------
// the full re-bin's scatter, and the placement of the last step's arrivals
// ---------------------------------------------------------------------------
template <class T>
__device__ __forceinline__ void put_slot(const View<T> &V, int64_t q, const MoverRec<T> &r)
{
    V.ox[q] = r.ox;
    V.oy[q] = r.oy;
    V.oz[q] = r.oz;
    V.vx[q] = r.vx;
    V.vy[q] = r.vy;
    V.vz[q] = r.vz;
    V.d[q] = r.d;
    V.id[q] = r.id;
}

// Records in a store's arrays: seven arrays of slots T, each a run of slots / 8
// records of eight T, together at least 7/8 * 5/4 of the capacity.
template <class T>
struct RecordArrays {
    View<T> W;
    int64_t per;   // records per array

    __device__ __forceinline__ RecordArrays(const View<T> &v, int64_t slots) : W(v), per(slots / 8)
    {
    }
    __device__ __forceinline__ MoverRec<T> *at(int64_t k) const
    {
        T *const a[7] = {W.ox, W.oy, W.oz, W.vx, W.vy, W.vz, W.d};
        T *b = a[0];
        int64_t j = k;
#pragma unroll
        for (int i = 1; i < 7; ++i)
            if (k >= i * per) {
                b = a[i];
                j = k - i * per;
            }
        return reinterpret_cast<MoverRec<T> *>(b) + j;
    }
};

// Where injections are staged until a full re-bin places them: memory of their
// own, or, while no particle has been placed, the empty store's arrays,
// which hold them all, so that a first load in one call takes one re-bin (3e6
// droplets: 0.45 to 0.12 ms).  Their chunks beside them (the store's id array).
// Nothing of the store, its containers or its inboxes is written for them: a
// read-out of the store may still run on another stream, and a captured step may
// be replayed before they are placed.
template <class T>
struct Staging {
    Views<T> V;
    const int32_t *flags;
    MoverRec<T> *rec;
    int32_t *dest;
    int64_t slots;
    int32_t in_store;
};
template <class T>
struct StagingAt {
    RecordArrays<T> own;
    MoverRec<T> *rec;
    int32_t *dest;
    bool in_store;
    __device__ __forceinline__ explicit StagingAt(const Staging<T> &s)
        : own(s.V.pick(s.flags[F_CUR]), s.slots), rec(s.rec), in_store(s.in_store != 0)
    {
        dest = in_store ? own.W.id : s.dest;
    }
    __device__ __forceinline__ MoverRec<T> *at(int64_t k) const
    {
        return in_store ? own.at(k) : rec + k;
    }
};

template <class T>
struct ScatterArgs {
    Views<T> V;
    const Cont *cont0, *cont1;
    const MoverRec<T> *rec;  // inboxes [2][nrec]
    int64_t nrec;
    Staging<T> staged;
    int64_t npend;           // staged injections
    const int4 *lay;
    int32_t *cursor;
    int32_t *flags;
    int64_t C;
    InboxRule inbox;
    int32_t sparse;          // containers hold few particles: a wave for each
    Params p;
    int4 *src;               // sources, and a chunk's size in 16-byte pieces
    int32_t src_pieces;
    int32_t *written;
};

// the slot of a chunk's particle number `rank` in the new layout
__device__ __forceinline__ int64_t slot_of_rank(const int4 &l, int32_t rank)
{
    const int32_t i = rank < l.y ? 0 : rank / l.y;
    return (int64_t)l.x + (int64_t)i * l.z + (rank - i * l.y);
}

// 512 threads: larger tiles take fewer reservations of a crowded chunk and
// leave fewer partial lines, smaller workgroups hide more latency (tiles of
// 2048, 4096 and, with 512 and 1024 threads, 8192 and 16384 droplets: 321, 203,
// 187 and 211 us of scatter for 3e6; a re-bin of 4e8: 28.0 ms at 256 threads,
// 25.2 at 512, 29.3 at 1024).
constexpr int kScatterBlock = 512;
constexpr int kScatterGroups = 1024;   // they run every step and usually exit at the gate

// Staged injections per chunk are counted, and placed, in tiles of kTile per
// workgroup through LDS counters of every chunk while there are at most
// kHistMax chunks, so that the counter of a crowded chunk is taken once per
// tile: device atomics on one address are served one after the other (8 x
// 375e3 droplets in two plumes on 1728 chunks: 8 x 0.53 ms of counts and 8 x
// 0.57 ms of scatters with an atomic per droplet, 16 and 187 us in all now; on
// 8000 chunks, putting in 3e6 uniform droplets 0.74 against 1.16 ms, in two plumes
// 0.50 against 3.7, 3e5 uniform ones 0.34 against 0.36).  More chunks than these do
// not fit 32 KB of LDS, and their counters are less crowded: a droplet takes its
// own atomic.
constexpr int kHistMax = 8192;
constexpr int kTilePer = 16, kTile = kTilePer * kScatterBlock;

// Containers of more slots than kWaveSlots are never a wave's, up to kBigMax of a
// workgroup's (a wave takes 64 slots in the time of a workgroup's 512).
constexpr int kWaveSlots = 1024, kBigMax = 256;

// Full re-bin: the occupied slots and the records, chunk by chunk, into the
// second store, which the last workgroup makes the store.  A container's
// particles that stay in its chunk get the consecutive places that the layout
// set for them, and so do its arrivals.  A workgroup takes a container at a
// time, or, where they hold few particles (`sparse`), each of its waves does: the
// time of a small container is latency (an injection of 1000 and a step of 1e6
// droplets in 32 768 containers 588 us by workgroups, 380 by waves; of 1e5 in
// 32 768, 440 and 257).
template <class T>
__global__ void __launch_bounds__(kScatterBlock) k_scatter(ScatterArgs<T> a)
{
    if (!a.flags[F_GO]) return;
    __shared__ int32_t pos, nbig, big[kBigMax], hist[kHistMax];
    __shared__ bool last;
    const int cur = a.flags[F_CUR], t = a.flags[F_TICK];
    const int32_t ni = cur ? a.flags[F_NITEMS1] : a.flags[F_NITEMS];
    const View<T> V = a.V.pick(cur), W = a.V.pick(cur ^ 1);
    const Cont *const ct = cur ? a.cont1 : a.cont0;
    const int m = (t + 2) % 3;
    const MoverRec<T> *const rec = a.rec + ((t + 1) & 1) * a.nrec;
    // Moves the slots first, first + step, ... of a container (lanes' slots
    // consecutive) and its inbox's records; take(n) reserves places of those that stay.
    auto move = [&](int32_t it, const ContState &me, int32_t nin, int32_t first, int32_t step,
                    auto take) {
        const int32_t c = me.c, cnt = me.cnt;
        const int4 l = a.lay[c];
        const int32_t in0 = ct[it].place[1];
        for (int32_t o1 = first; o1 - (int32_t)__lane_id() < cnt; o1 += step) {   // every lane
            const int64_t q = (int64_t)me.base + o1;
            MoverRec<T> r;
            int64_t cn = -1;
            bool home = false;
            if (o1 < cnt) {
                r = MoverRec<T>{V.ox[q], V.oy[q], V.oz[q], V.vx[q], V.vy[q], V.vz[q], V.d[q],
                                V.id[q]};
                if (occupied(r.ox, r.d)) {
                    // (a particle can leave its chunk and still be in it: one
                    // chunk along a periodic axis)
                    home = !a.p.global && !left_chunk(r.ox, r.oy, r.oz, T(a.p.E));
                    cn = home ? c : chunk_of_stored(a.p, c, r.ox, r.oy, r.oz);
                    home = home || (a.p.global && cn == c);
                }
            }
            const uint64_t stay = __ballot(home);
            const int32_t b = take(__popcll(stay));
            if (home)
                put_slot(W, slot_of_rank(l, b + __popcll(stay & lanes_below_mask())), r);
            else if (cn >= 0)   // a mover whose inbox was full
                put_slot(W, slot_of_rank(a.lay[cn], atomicAdd(&a.cursor[cn], 1)), r);
        }
        for (int32_t r = first; r < nin; r += step)
            put_slot(W, slot_of_rank(l, in0 + r), rec[me.ibase + r]);
    };
    auto arrivals = [&](const ContState &me) { return min(me.in, inbox_cap(me.room, a.inbox)); };
    auto by_workgroup = [&](int32_t it) {
        const ContState me = state_of(ct + it, m);
        const int32_t nin = arrivals(me);
        if (me.cnt == 0 && nin == 0) return;   // uniform
        if (threadIdx.x == 0) pos = ct[it].place[0];
        __syncthreads();
        move(it, me, nin, threadIdx.x, kScatterBlock, [&](int32_t n) {
            int32_t b = 0;
            if (__lane_id() == 0) b = n ? atomicAdd(&pos, n) : 0;
            return __shfl(b, 0);
        });
        __syncthreads();
    };
    if (a.sparse) {
        // a container per wave, those of more slots than kWaveSlots left to the
        // workgroup (as many as it can note)
        if (threadIdx.x == 0) nbig = 0;
        __syncthreads();
        const int32_t waves = kScatterBlock / 64;
        for (int32_t w = blockIdx.x * waves + (threadIdx.x >> 6); w < ni; w += gridDim.x * waves) {
            const int32_t it = __builtin_amdgcn_readfirstlane(w);
            const ContState me = state_of(ct + it, m);
            const int32_t nin = arrivals(me);
            if (me.cnt == 0 && nin == 0) continue;
            if (me.cnt > kWaveSlots) {
                int32_t k = 0;
                if (__lane_id() == 0) k = atomicAdd(&nbig, 1);
                k = __shfl(k, 0);
                if (k < kBigMax) {
                    if (__lane_id() == 0) big[k] = it;
                    continue;
                }
            }
            int32_t at = ct[it].place[0];
            move(it, me, nin, __lane_id(), 64, [&](int32_t n) {
                at += n;
                return at - n;
            });
        }
        __syncthreads();
        const int32_t nb = min(nbig, kBigMax);
        for (int32_t k = 0; k < nb; ++k) by_workgroup(big[k]);
    } else {
        for (int32_t it = blockIdx.x; it < ni; it += gridDim.x) by_workgroup(it);
    }
    const StagingAt<T> staged(a.staged);
    for (int64_t r0 = (int64_t)blockIdx.x * kTile; r0 < a.npend;
         r0 += (int64_t)gridDim.x * kTile) {
        int32_t cn[kTilePer], rank[kTilePer];
        if (a.C <= kHistMax) {
            __syncthreads();
            for (int32_t i = threadIdx.x; i < a.C; i += kScatterBlock) hist[i] = 0;
            __syncthreads();
        }
#pragma unroll
        for (int j = 0; j < kTilePer; ++j) {
            const int64_t r = r0 + j * kScatterBlock + threadIdx.x;
            cn[j] = r < a.npend ? staged.dest[r] : -1;
            rank[j] = cn[j] < 0 ? 0
                                : atomicAdd(a.C <= kHistMax ? &hist[cn[j]] : &a.cursor[cn[j]], 1);
        }
        if (a.C <= kHistMax) {
            __syncthreads();
            // a thread's reservations are in flight together, and the
            // workgroups start at different chunks
            const int32_t C = (int32_t)a.C;
            const int32_t rot = (int32_t)((int64_t)(r0 / kTile) * 97 % C);
            constexpr int kBatch = 8;
            for (int32_t i0 = threadIdx.x; i0 < C; i0 += kBatch * kScatterBlock) {
                int32_t h[kBatch], at[kBatch];
#pragma unroll
                for (int k = 0; k < kBatch; ++k) {
                    const int32_t i = i0 + k * kScatterBlock;
                    at[k] = i < C ? (i + rot < C ? i + rot : i + rot - C) : -1;
                    h[k] = at[k] < 0 ? 0 : hist[at[k]];
                }
#pragma unroll
                for (int k = 0; k < kBatch; ++k)
                    if (h[k]) h[k] = atomicAdd(&a.cursor[at[k]], h[k]);
#pragma unroll
                for (int k = 0; k < kBatch; ++k)
                    if (at[k] >= 0) hist[at[k]] = h[k];
            }
            __syncthreads();
        }
#pragma unroll
        for (int j = 0; j < kTilePer; ++j) {
            if (cn[j] < 0) continue;
            if (a.C <= kHistMax) rank[j] += hist[cn[j]];
            put_slot(W, slot_of_rank(a.lay[cn[j]], rank[j]),
                     *staged.at(r0 + j * kScatterBlock + threadIdx.x));
        }
    }
    // a chunk of several containers adds to its sources atomically: those that
    // are only marked as cleared become zeros
    for (int64_t c = (int64_t)blockIdx.x * kScatterBlock + threadIdx.x; c < a.C;
         c += (int64_t)gridDim.x * kScatterBlock) {
        if (a.lay[c].w == 1 || a.written[c]) continue;
        for (int32_t i = 0; i < a.src_pieces; ++i) a.src[c * a.src_pieces + i] = int4{0, 0, 0, 0};
        a.written[c] = 1;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        last = atomicAdd(&a.flags[F_TICKET], 1) == (int32_t)gridDim.x - 1;
        if (last) {   // every workgroup has passed the gate and read the flags
            a.flags[F_CUR] = cur ^ 1;
            a.flags[F_GO] = 0;
            a.flags[F_REPACKS] += 1;
        }
    }
}

// Places the last step's arrivals, as the next step's kernel would (for
// calls that need the store whole): into the holes, then past the last slot.
template <class T>
__global__ void __launch_bounds__(256) k_settle(Views<T> VV, Cont *cont0, Cont *cont1,
                                                const MoverRec<T> *recs, int64_t nrec,
                                                int32_t *flags, int32_t *spread)
{
    __shared__ int32_t apop;
    const int cur = flags[F_CUR], t = flags[F_TICK];
    const int32_t ni = cur ? flags[F_NITEMS1] : flags[F_NITEMS];
    const View<T> V = VV.pick(cur);
    Cont *const ct = cur ? cont1 : cont0;
    const int m = (t + 2) % 3;
    const MoverRec<T> *const rec = recs + ((t + 1) & 1) * nrec;
    for (int32_t it = blockIdx.x; it < ni; it += gridDim.x) {
        const ContState me = state_of(ct + it, m);
        const int32_t n_in = me.in;
        if (n_in == 0) continue;   // uniform
        const int32_t nq_old = me.cnt, h = me.h;
        const int32_t nq = nq_old + max(0, n_in - h);
        __syncthreads();
        if (threadIdx.x == 0) apop = 0;
        __syncthreads();
        for (int32_t o = threadIdx.x; o < nq; o += 256) {
            const int64_t q = (int64_t)me.base + o;
            if (o < nq_old && occupied(V.ox[q], V.d[q])) continue;
            const int32_t r = atomicAdd(&apop, 1);
            if (r < n_in) put_slot(V, q, rec[me.ibase + r]);
        }
        if (threadIdx.x == 0) {
            ct[it].in[m] = 0;
            ct[it].s[m] = {nq, max(0, h - n_in)};
            atomicAdd(&spread[16 * (it % kSpread)], max(0, h - n_in) - h);
        }
    }
}

// non-empty containers and holes (as they are once the arrivals are placed)
__global__ void __launch_bounds__(256) k_stats(const Cont *cont0, const Cont *cont1,
                                               int32_t *flags)
{
    const int cur = flags[F_CUR], t = flags[F_TICK];
    const int32_t ni = cur ? flags[F_NITEMS1] : flags[F_NITEMS];
    const Cont *const ct = cur ? cont1 : cont0;
    const int m = (t + 2) % 3;
    int32_t items = 0, holes = 0;
    for (int32_t j = blockIdx.x * 256 + threadIdx.x; j < ni; j += gridDim.x * 256) {
        const int32_t in = ct[j].in[m];
        items += ct[j].s[m].cnt - ct[j].s[m].h + in > 0;
        holes += max(0, ct[j].s[m].h - in);
    }
    for (int o = 32; o > 0; o >>= 1) {
        items += __shfl_xor(items, o);
        holes += __shfl_xor(holes, o);
    }
    if (__lane_id() == 0) {
        atomicAdd(&flags[F_STAT_ITEMS], items);
        atomicAdd(&flags[F_STAT_HOLES], holes);
    }
}

// the runs of a settled store's containers
__global__ void __launch_bounds__(256) k_runs(const Cont *cont0, const Cont *cont1,
                                              const int32_t *flags, RunItem *items,
                                              int32_t *nitems)
{
    const int cur = flags[F_CUR], t = flags[F_TICK];
    const int32_t ni = cur ? flags[F_NITEMS1] : flags[F_NITEMS];
    const Cont *const ct = cur ? cont1 : cont0;
    const int m = (t + 2) % 3;
    if (blockIdx.x == 0 && threadIdx.x == 0) *nitems = ni;
    for (int32_t j = blockIdx.x * 256 + threadIdx.x; j < ni; j += gridDim.x * 256)
        items[j] = RunItem{ct[j].c, ct[j].base, ct[j].s[m].cnt, ct[j].k};
}

// ---------------------------------------------------------------------------
// inject: binary64 global positions -> chunk + chunk-local offsets, staged
// ---------------------------------------------------------------------------
template <class T>
__global__ void k_stage(int64_t n, const double *x, const double *up, const double *d,
                        int64_t at, int64_t id0, Params p, Staging<T> to, int32_t *flags)
{
    const StagingAt<T> staged(to);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        bool ok = true;
        int64_t ch[3];
        T loc[3];
        for (int a = 0; a < 3; ++a) {
            double xa = x[3 * i + a];
            if (!isfinite(xa)) { ok = false; xa = 0.0; }
            // periodic image in [0, L)
            xa = xa - floor(xa / p.L[a]) * p.L[a];
            if (xa >= p.L[a] || xa < 0.0) xa = 0.0;
            if (p.global) {   // binary32 metres; its cell from the binary32 product
                float xf = (float)xa;
                if (xf >= p.Lf[a]) xf = 0.f;
                ch[a] = gcell(xf, p.inv_hf[a], p.n[a]) / p.E;
                loc[a] = (T)xf;
                continue;
            }
            double g = xa / p.h[a];                  // cell units
            int64_t ci = (int64_t)floor(g);
            if (ci >= p.n[a]) { g -= p.n[a]; ci -= p.n[a]; }
            if (ci < 0) { g += p.n[a]; ci += p.n[a]; }
            ch[a] = ci / p.E;
            T o = (T)(g - (double)(ch[a] * p.E));   // exact before the rounding to T
            const int k = rebase(o, T(p.E), T(1) / T(p.E));
            ch[a] = wrapi(ch[a] + k, p.nc[a]);
            loc[a] = o;
        }
        const double v[3] = {up[3 * i], up[3 * i + 1], up[3 * i + 2]};
        const double dd = d[i];
        for (int a = 0; a < 3; ++a)
            if (!isfinite(v[a])) ok = false;
        if (!isfinite(dd) || !(dd > 0.0)) ok = false;
        const int64_t m = at + i;
        *staged.at(m) = MoverRec<T>{loc[0], loc[1], loc[2], (T)v[0], (T)v[1], (T)v[2], (T)dd,
                                (int32_t)(id0 + i)};
        // (a diameter that the state's precision rounds to zero is accepted,
        // but no slot can hold it)
        staged.dest[m] =
            ok && (T)dd > T(0) ? (int32_t)chunk_index(p, ch[0], ch[1], ch[2]) : -1;
        if (!ok) flags[F_BADINPUT] = 1;
    }
}

// Counts the staged injections of each chunk (for the layout of the full
// re-bin that places them).  Those without a chunk (a bad value in a batch that
// was staged in parts) are neither counted nor placed.
template <class T>
__global__ void __launch_bounds__(kScatterBlock) k_count_staged(int32_t *staged,
                                                                int64_t stride, Staging<T> from,
                                                                int64_t at, int64_t n, int64_t C)
{
    __shared__ int32_t hist[kHistMax];
    const int32_t *const dest = StagingAt<T>(from).dest + at;
    const bool lds = C <= kHistMax;
    if (lds) {
        for (int32_t i = threadIdx.x; i < C; i += kScatterBlock) hist[i] = 0;
        __syncthreads();
    }
    for (int64_t i = (int64_t)blockIdx.x * kScatterBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kScatterBlock)
        if (dest[i] >= 0) atomicAdd(lds ? &hist[dest[i]] : &staged[dest[i] * stride], 1);
    if (lds) {
        __syncthreads();
        for (int32_t i = threadIdx.x; i < C; i += kScatterBlock)
            if (hist[i]) atomicAdd(&staged[i * stride], hist[i]);
    }
}

// ---------------------------------------------------------------------------
// outputs
// ---------------------------------------------------------------------------
// Where the read-out goes (any may be null); particle k's row k of each.
struct ParticleOut {
    double *x, *up, *d;
    int64_t *id;
    int32_t *cell;
};

// Writes particle k of chunk c with stored position o, velocity v, diameter dd.
template <class T>
__device__ __forceinline__ void put_particle(const ParticleOut &out, const Params &p, int64_t k,
                                             int64_t c, const T (&o)[3], const T (&v)[3], T dd)
{
    const int32_t cc[3] = {(int32_t)(c % p.nc[0]), (int32_t)((c / p.nc[0]) % p.nc[1]),
                           (int32_t)(c / ((int64_t)p.nc[0] * p.nc[1]))};
    for (int a = 0; a < 3; ++a) {
        const double org = (double)((int64_t)cc[a] * p.E);
        if (p.global) {   // binary32 metres
            if (out.x) out.x[3 * k + a] = (double)o[a];
            if (out.cell) out.cell[3 * k + a] = gcell((float)o[a], p.inv_hf[a], p.n[a]);
        } else {
            if (out.x) out.x[3 * k + a] = (org + (double)o[a]) * p.h[a];
            if (out.cell)
                out.cell[3 * k + a] = cc[a] * p.E + min(max((int)o[a], 0), p.E - 1);
        }
        if (out.up) out.up[3 * k + a] = (double)v[a];
    }
    if (out.d) out.d[k] = (double)dd;
    if (out.id) out.id[k] = k;
}

// Calls f(chunk, record) for every particle: the occupied slots of the
// containers' runs and the arrivals waiting in their inboxes.
template <class T, class F>
__device__ __forceinline__ void each_particle(const Current<T> &S, const F &f)
{
    const View<T> &V = S.V;
    for (int32_t it = blockIdx.x; it < S.ni; it += gridDim.x) {
        const ContState me = state_of(S.cont + it, S.m);
        for (int32_t o = threadIdx.x; o < me.cnt; o += blockDim.x) {
            const int64_t q = (int64_t)me.base + o;
            const MoverRec<T> r{V.ox[q], V.oy[q], V.oz[q], V.vx[q], V.vy[q], V.vz[q], V.d[q],
                                V.id[q]};
            if (occupied(r.ox, r.d)) f(me.c, r);
        }
        for (int32_t j = threadIdx.x; j < me.in; j += blockDim.x)
            f(me.c, S.rec[me.ibase + j]);
    }
}

// Read-out straight from the store: a particle's row of each output lies
// wherever its id does, so each is a partial-line write.
template <class T>
__global__ void __launch_bounds__(256) k_get_particles(Store<T> st, Params p, int64_t count,
                                                       ParticleOut out)
{
    const Current<T> S(st);
    each_particle(S, [&](int32_t c, const MoverRec<T> &r) {
        if (r.id < 0 || r.id >= count) return;   // never in a consistent store
        const T o[3] = {r.ox, r.oy, r.oz};
        const T v[3] = {r.vx, r.vy, r.vz};
        put_particle<T>(out, p, r.id, c, o, v, r.d);
    });
}

// Read-out of many particles in two passes: one scattered write per particle
// (its record with its chunk, by id), then the records in id order into the
// outputs, whole lines at a time.  The records lie in the re-bin's second
// store, which holds nothing between re-bins.  1e7 binary32 particles, all
// outputs: 0.67 ms (0.075 ms clearing, 0.38 ms the scattered records, 0.22 ms
// out), against 2.06 ms directly.
template <class T>
__global__ void __launch_bounds__(256) k_records_clear(Store<T> st, int64_t slots, int64_t count)
{
    const RecordArrays<T> r(st.V.pick(st.flags[F_CUR] ^ 1), slots);
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < count) *r.at(k) = MoverRec<T>{T(0), T(0), T(0), T(0), T(0), T(0), T(0), -1};
}

template <class T>
__global__ void __launch_bounds__(256) k_records_by_id(Store<T> st, int64_t slots, int64_t count)
{
    const RecordArrays<T> to(st.V.pick(st.flags[F_CUR] ^ 1), slots);
    const Current<T> S(st);
    each_particle(S, [&](int32_t c, MoverRec<T> r) {
        const int64_t k = r.id;
        if (k < 0 || k >= count) return;
        r.id = c;
        *to.at(k) = r;
    });
}

// A workgroup's 256 rows of the [count][3] outputs pass through LDS, so that
// the lanes' stores are consecutive.
template <class T>
__global__ void __launch_bounds__(256) k_records_out(Store<T> st, int64_t slots, Params p,
                                                     int64_t count, ParticleOut out)
{
    __shared__ double sx[768], su[768];
    __shared__ int32_t sc[768];
    __shared__ int there[256];
    const RecordArrays<T> r(st.V.pick(st.flags[F_CUR] ^ 1), slots);
    const int64_t k0 = (int64_t)blockIdx.x * 256;
    const int64_t k = k0 + threadIdx.x;
    MoverRec<T> m;
    m.id = -1;
    if (k < count) m = *r.at(k);
    there[threadIdx.x] = m.id >= 0;   // else no slot holds it (never in a consistent store)
    if (m.id >= 0) {
        const T o[3] = {m.ox, m.oy, m.oz};
        const T v[3] = {m.vx, m.vy, m.vz};
        const ParticleOut rows{sx, su, nullptr, nullptr, sc};
        put_particle<T>(rows, p, threadIdx.x, m.id, o, v, m.d);
        if (out.d) out.d[k] = (double)m.d;
        if (out.id) out.id[k] = k;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int e = threadIdx.x + 256 * j;
        if (!there[e / 3]) continue;
        if (out.x) out.x[3 * k0 + e] = sx[e];
        if (out.up) out.up[3 * k0 + e] = su[e];
        if (out.cell) out.cell[3 * k0 + e] = sc[e];
    }
}

// Chunk-major sources into the field layout, and their reset.  A workgroup
// takes the chunks of 32 cells along x (one chunk along y and z), 16 lanes a
// row of cell pairs, its loads issued before its stores: its stores are rows of
// 256 bytes and what it reads of a chunk is consecutive.  A reset only marks
// the chunks as cleared (the next step stores over them instead of adding, and
// a read-out of a marked chunk is zeros without reading); chunks of several
// containers, which add atomically, are set to zero.
// Bound by HBM (16 B a value).  With reset, 128^3 cells in 15.9 us, 256^3 in
// 0.10 ms, 512^3 in 1.22 ms, where reading, writing and clearing every value in
// the layout of the output took 21.9 us, 0.26 and 2.1 ms; the step saves the
// read of the cleared sources besides (12 KB a chunk).
constexpr int kSrcCells = 32;
template <class A, int E>
__global__ void __launch_bounds__(256) k_get_sources(A *src, int32_t *written, const int32_t *first0,
                                                     const int32_t *first1, const int32_t *flags,
                                                     Params p, double *out, int reset)
{
    typedef A pair __attribute__((ext_vector_type(2)));
    typedef double dpair __attribute__((ext_vector_type(2)));
    constexpr int E3 = E * E * E, NC = kSrcCells / E;
    constexpr int rows = 3 * E * E, NR = (rows + 15) / 16;
    const int32_t nbx = (p.nc[0] + NC - 1) / NC;
    const int64_t runs = (int64_t)nbx * p.nc[1] * p.nc[2];
    const int lane = threadIdx.x & 15, r0 = threadIdx.x >> 4;
    const int ch = 2 * lane / E, i = 2 * lane % E;      // chunk of the run, cell in it
    const int32_t *const first = flags[F_CUR] ? first1 : first0;
    const bool whole = ((uintptr_t)out & 15) == 0;
    for (int64_t run = blockIdx.x; run < runs; run += gridDim.x) {
        const int64_t b = run / nbx;
        const int32_t cx0 = (int32_t)(run - b * nbx) * NC;
        const int32_t cz = (int32_t)(b / p.nc[1]), cy = (int32_t)(b - (int64_t)cz * p.nc[1]);
        const int64_t c0 = b * p.nc[0] + cx0;
        const bool in = cx0 + ch < p.nc[0];
        const bool have = in && written[c0 + ch] != 0;
        const bool several = in && reset && first[c0 + ch + 1] - first[c0 + ch] > 1;
        pair v[NR];
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            const int r = r0 + 16 * u;   // (comp, k, j)
            v[u] = pair{A(0), A(0)};
            if (have && r < rows) v[u] = *(const pair *)(src + (c0 + ch) * 3 * E3 + r * E + i);
        }
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            const int r = r0 + 16 * u;
            if (!in || r >= rows) continue;
            const int comp = r / (E * E), k = r / E % E, j = r % E;
            double *o = out + ((((int64_t)comp * p.n[2] + cz * E + k) * p.n[1] + cy * E + j) *
                                   p.n[0] + cx0 * E + 2 * lane);
            const dpair w = {(double)v[u][0], (double)v[u][1]};
            if (whole) {
                *(dpair *)o = w;
            } else {
                o[0] = w[0];
                o[1] = w[1];
            }
            if (several && have) *(pair *)(src + (c0 + ch) * 3 * E3 + r * E + i) = pair{A(0), A(0)};
        }
        if (!reset) continue;
        __syncthreads();   // every thread has read the marks
        if (r0 == 0 && i == 0 && have && !several) written[c0 + ch] = 0;
    }
}

__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// synthetic fluid update: U^k = R_z(theta_k) U^0, rounded once to T
template <class T>
__global__ void k_rotate(const T *u0, T *u, int64_t ncell, double cs, double sn)
{
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < ncell;
         q += (int64_t)gridDim.x * blockDim.x) {
        const double ux = (double)u0[q], uy = (double)u0[ncell + q];
        u[q] = (T)(cs * ux - sn * uy);
        u[ncell + q] = (T)(sn * ux + cs * uy);
        u[2 * ncell + q] = u0[2 * ncell + q];
    }
}

// checkpoint copy of the (settled) store, all slots, and its containers; or
// back (into the current store, whichever of the two it is by then)
template <class T>
__global__ void k_snapshot(Views<T> VV, Cont *cont0, Cont *cont1, int32_t *first0,
                           int32_t *first1, int64_t slots, int64_t C, char *buf, SnapLayout L,
                           int32_t *flags, int32_t *spread, int restore)
{
    const int cur = flags[F_CUR], t = flags[F_TICK];
    const View<T> V = VV.pick(cur);
    Cont *const ct = cur ? cont1 : cont0;
    int32_t *const first = cur ? first1 : first0;
    const int m = (t + 2) % 3;
    T *arr[7] = {V.ox, V.oy, V.oz, V.vx, V.vy, V.vz, V.d};
    T *sT = reinterpret_cast<T *>(buf + L.state);
    int32_t *sid = reinterpret_cast<int32_t *>(buf + L.id);
    RunItem *sitems = reinterpret_cast<RunItem *>(buf + L.items);
    int32_t *snitems = reinterpret_cast<int32_t *>(buf + L.nitems);
    Cont *scont = reinterpret_cast<Cont *>(buf + L.cont);
    int32_t *sfirst = reinterpret_cast<int32_t *>(buf + L.first);
    int32_t *const nitems = flags + (cur ? F_NITEMS1 : F_NITEMS);
    const int64_t g0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t gs = (int64_t)gridDim.x * blockDim.x;
    const int32_t ni = restore ? *snitems : *nitems;
    for (int64_t q = g0; q < slots; q += gs) {
        if (restore) {
            for (int a = 0; a < 7; ++a) arr[a][q] = sT[a * slots + q];
            V.id[q] = sid[q];
        } else {
            for (int a = 0; a < 7; ++a) sT[a * slots + q] = arr[a][q];
            sid[q] = V.id[q];
        }
    }
    for (int64_t j = g0; j < ni; j += gs) {
        const ContState me = state_of((restore ? scont : ct) + j, restore ? 0 : m);
        const int32_t cnt = me.cnt, h = me.h;
        const int at = restore ? m : 0;    // a saved container's state is its first
        Cont d = {};
        d.c = me.c;
        d.base = me.base;
        d.room = me.room;
        d.ibase = me.ibase;
        d.k = me.k;
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            d.s[u].cnt = u == at ? cnt : 0;
            d.s[u].h = u == at ? h : 0;
        }
        if (restore) {
            ct[j] = d;
            if (h) atomicAdd(&spread[16 * (j % kSpread)], h);   // (cleared before)
        } else {
            scont[j] = d;
            sitems[j] = RunItem{d.c, d.base, cnt, d.k};
        }
    }
    for (int64_t c = g0; c <= C; c += gs) {
        if (restore) first[c] = sfirst[c];
        else sfirst[c] = first[c];
    }
    if (g0 == 0) *(restore ? nitems : snitems) = ni;
}

// ---------------------------------------------------------------------------
// host-side helpers
// ---------------------------------------------------------------------------
inline int64_t grid_for(int64_t n, int64_t cap = 8192)
{
    int64_t g = (n + 255) / 256;
    if (g < 1) g = 1;
    return g > cap ? cap : g;
}

template <class F>
hipError_t dispatch(st_ctx *c, F &&f)
{
    switch (c->form) {
    case ST_FORM_FP64: return f(double(0), double(0));
    case ST_FORM_FP32_LOCAL: return f(float(0), double(0));
    default: return f(float(0), float(0));
    }
}

// ev[0], ev[1] (when not null) take the start and end of the kernel's own
// execution (not of the commands around it)
template <class T, class A, int E, int I, int D, int NB>
hipError_t launch_step_n(st_ctx *c, const StepArgs<T, A> &a, hipStream_t s, hipEvent_t *ev)
{
    const int64_t round = 8 * kXcdBlock;
    const int64_t grid = (c->max_items + round - 1) / round * round;
    if constexpr (sizeof(A) == 8) {   // only the forms that tape save
        if (a.sv[0]) {
            if (ev[0])
                hipExtLaunchKernelGGL((k_step<T, A, E, I, D, true, NB>), dim3(grid), dim3(NB), 0,
                                      s, ev[0], ev[1], 0, a);
            else
                hipLaunchKernelGGL((k_step<T, A, E, I, D, true, NB>), dim3(grid), dim3(NB), 0, s,
                                   a);
            return hipGetLastError();
        }
    }
    if (ev[0])
        hipExtLaunchKernelGGL((k_step<T, A, E, I, D, false, NB>), dim3(grid), dim3(NB), 0, s,
                              ev[0], ev[1], 0, a);
    else
        hipLaunchKernelGGL((k_step<T, A, E, I, D, false, NB>), dim3(grid), dim3(NB), 0, s, a);
    return hipGetLastError();
}

template <class T, class A, int E, int I, int D>
hipError_t launch_step_t(st_ctx *c, const StepArgs<T, A> &a, hipStream_t s, hipEvent_t *ev)
{
    // Twice the threads where the containers fill at most half of the 256 CUs
    // and hold more than one pass of 256 threads (32^3 mesh, 1e5 droplets in
    // binary64: 24.7 against 27.4 us a step with its sources; 100 containers of
    // 1600 droplets 18.8 against 21.3, in binary32 15.2 against 17.6).  Not with
    // 270 containers in the FP32-everywhere form (3 % slower).  Between the two the
    // line could lie higher: 125 to 252 containers of 800 to 4000 droplets are 8 to
    // 20 % faster with twice the threads in the other forms.
    // Half the threads on large meshes of sparse small chunks: a workgroup's time
    // is latency there, and twice as many are in flight (64^3 cells in chunks of
    // 2^3, 1 and 8 droplets a chunk in binary32: 196 -> 141 and 275 -> 189 us; 128^3,
    // 2 a chunk, 1.48 -> 0.91 ms; 192^3 in chunks of 4^3, 10 a chunk, 0.75 -> 0.50
    // ms).  Above that plumes' chunks can be crowded (64^3 in chunks of 2^3, 40 a
    // chunk, most in one plume: 293 -> 311 us; 64^3 in chunks of 4^3, 300 a chunk,
    // 131 -> 222), and meshes of fewer chunks are soon through.  The
    // FP32-everywhere form (whose state takes the most registers) gains longer: 40
    // and 60 a chunk 0.375 -> 0.24 and 0.36 -> 0.23 ms, in a plume 0.36 -> 0.37 and
    // 0.36 -> 0.33.
    if constexpr (E < 8)
        if (c->C >= 32768 && c->count <= c->C * (sizeof(A) == 4 ? 64 : 12))
            return launch_step_n<T, A, E, I, D, 128>(c, a, s, ev);
    if constexpr (E == 8)
        if (c->max_items <= 128 && c->count > c->C * 256 * (16 / (int64_t)sizeof(T)))
            return launch_step_n<T, A, E, I, D, 512>(c, a, s, ev);
    return launch_step_n<T, A, E, I, D, 256>(c, a, s, ev);
}

template <class T, class A, int E, int I>
hipError_t launch_step_d(st_ctx *c, const StepArgs<T, A> &a, hipStream_t s, hipEvent_t *ev)
{
    return c->prm.drag == 1 ? launch_step_t<T, A, E, I, 1>(c, a, s, ev)
                            : launch_step_t<T, A, E, I, 0>(c, a, s, ev);
}

template <class T, class A, int E>
hipError_t launch_step_e(st_ctx *c, const StepArgs<T, A> &a, hipStream_t s, hipEvent_t *ev)
{
    return c->prm.interp == 1 ? launch_step_d<T, A, E, 1>(c, a, s, ev)
                              : launch_step_d<T, A, E, 0>(c, a, s, ev);
}

template <class T>
Staging<T> staging_of(st_ctx *c)
{
    return Staging<T>{views_of<T>(c), c->flags, (MoverRec<T> *)c->stage, c->stage_dest, c->slots,
                      c->stage_in_store};
}

// Up to this many chunks the gate's own workgroup makes the layout.  Behind a
// step the three launches of the other way nearly always find nothing to do and
// cost it 13 us all the same; behind injections there is always a layout to
// make (an injection placed and read: 3072 chunks 166 us in one workgroup, 177 in three
// launches, 4096 187 and 184, 6144 223 and 201).  Layout of 32768 chunks in one
// workgroup 0.27 ms against 0.031 in three launches, of 262144 2.3 ms against 0.048, of
// 2097152 20 ms against 0.23: at 32768 the launches pay from a full re-bin every 18
// steps on.
constexpr int64_t kLayoutOneStep = 32768, kLayoutOneFlush = 4096;

// The scatter's containers are taken by waves up to this many particles for each
// on the average (placing an injection, 40 a container 0.67 by workgroups and 0.49
// ms by waves, in a plume 0.73 and 0.56; 100 a container 0.205 and 0.182, but in a
// plume 0.227 and 0.262).
constexpr int64_t kSparsePer = 64;

// everything after the step kernel (or, npend > 0, the placing of the staged
// injections): the gate, and the full re-bin's scatter
template <class T>
hipError_t launch_rebin(st_ctx *c, int64_t npend, hipStream_t s)
{
    wrote_store(c, s);
    const bool one = c->C <= (npend ? kLayoutOneFlush : kLayoutOneStep);
    const GateArgs g{c->cont[0], c->cont[1], c->first[0], c->first[1], c->new_cnt, c->cursor,
                     c->lay, c->flags, c->spread, c->lay_sums, c->lay_part, c->C,
                     {c->prm.nc[0], c->prm.nc[1], c->prm.nc[2]},
                     c->slots - (int64_t)kAlign * c->max_items, c->inbox, npend == 0,
                     npend ? c->staged : nullptr, c->staged_stride, one};
    hipLaunchKernelGGL(k_gate, dim3(1), dim3(1024), 0, s, g);
    if (!one) {
        const dim3 lb((c->C + kLayBlock - 1) / kLayBlock);
        hipLaunchKernelGGL(k_lay_count, lb, dim3(kLayBlock), 0, s, g);
        hipLaunchKernelGGL(k_lay_rooms, lb, dim3(kLayBlock), 0, s, g);
        hipLaunchKernelGGL(k_lay_write, lb, dim3(kLayBlock), 0, s, g);
    }
    const ScatterArgs<T> a{views_of<T>(c), c->cont[0], c->cont[1],
                           (const MoverRec<T> *)c->rec, c->nrec, staging_of<T>(c), npend, c->lay,
                           c->cursor, c->flags, c->C, c->inbox,
                           c->count + npend <= kSparsePer * c->max_items, c->prm,
                           (int4 *)c->src,
                           (int32_t)(3 * c->prm.E * c->prm.E * c->prm.E * c->asize / 16),
                           c->written};
    const int64_t n = std::max(c->max_items, npend / kTile);
    hipLaunchKernelGGL((k_scatter<T>), dim3(std::min<int64_t>(kScatterGroups, n)),
                       dim3(kScatterBlock), 0, s, a);
    return hipGetLastError();
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
namespace {
// no particles: a container without slots for every chunk
__global__ void k_init(Cont *cont, int32_t *first, int32_t *flags, int64_t C)
{
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c <= C;
         c += (int64_t)gridDim.x * blockDim.x) {
        first[c] = (int32_t)c;
        if (c < C) {
            Cont d = {};
            d.c = (int32_t)c;
            d.k = 1;
            cont[c] = d;
        }
        if (c == 0) flags[F_NITEMS] = (int32_t)C;
    }
}
}  // namespace

hipError_t launch_init(st_ctx *c, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(256), 0, s, c->flags, (int64_t)F_COUNT, 0);
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(kSpreadInts)), dim3(256), 0, s, c->spread,
                       (int64_t)kSpreadInts, 0);
    hipLaunchKernelGGL(k_init, dim3(grid_for(c->C + 1)), dim3(256), 0, s, c->cont[0], c->first[0],
                       c->flags, c->C);
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(c->C * c->staged_stride)), dim3(256), 0, s,
                       c->staged, c->C * c->staged_stride, 0);
    return hipGetLastError();
}

hipError_t launch_settle(st_ctx *c, hipStream_t s)
{
    wrote_store(c, s);
    return dispatch(c, [&](auto t, auto) -> hipError_t {
        using T = decltype(t);
        hipLaunchKernelGGL((k_settle<T>), dim3(std::min<int64_t>(c->max_items, 4096)), dim3(256), 0,
                           s, views_of<T>(c), c->cont[0], c->cont[1],
                           (const MoverRec<T> *)c->rec, c->nrec, c->flags, c->spread);
        return hipGetLastError();
    });
}

namespace {
template <class T>
hipError_t count_staged(st_ctx *c, int64_t at, int64_t n, hipStream_t s)
{
    if (n > 0) {
        const int64_t g = std::min<int64_t>((n + kTile - 1) / kTile, 512);
        hipLaunchKernelGGL((k_count_staged<T>), dim3(g), dim3(kScatterBlock), 0, s, c->staged,
                           c->staged_stride, staging_of<T>(c), at, n, c->C);
    }
    return hipGetLastError();
}
}  // namespace

hipError_t launch_stats(st_ctx *c, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, s, c->flags + F_STAT_ITEMS, (int64_t)2, 0);
    hipLaunchKernelGGL(k_stats, dim3(grid_for(c->max_items, 1024)), dim3(256), 0, s, c->cont[0],
                       c->cont[1], c->flags);
    return hipGetLastError();
}

hipError_t launch_runs(st_ctx *c, RunItem *items, int32_t *nitems, hipStream_t s)
{
    hipLaunchKernelGGL(k_runs, dim3(grid_for(c->max_items, 1024)), dim3(256), 0, s, c->cont[0],
                       c->cont[1], c->flags, items, nitems);
    return hipGetLastError();
}

hipError_t launch_step(st_ctx *c, const void *u, double dt, int deposit, hipStream_t s,
                       void *save)
{
    return dispatch(c, [&](auto t, auto acc) -> hipError_t {
        using T = decltype(t);
        using A = decltype(acc);
        StepArgs<T, A> a;
        a.V = views_of<T>(c);
        a.cont0 = c->cont[0];
        a.cont1 = c->cont[1];
        a.first0 = c->first[0];
        a.first1 = c->first[1];
        for (int k = 0; k < 7; ++k) a.sv[k] = nullptr;
        if (save) {
            const SnapLayout L = snap_layout(c->slots, c->tsize, c->C, c->max_items);
            char *b = (char *)save;
            for (int k = 0; k < 7; ++k) a.sv[k] = (T *)(b + L.state) + k * c->slots;
            a.sid = (int32_t *)(b + L.id);
            a.sitems = (RunItem *)(b + L.items);
            a.snitems = (int32_t *)(b + L.nitems);
        }
        a.u = (const T *)u;
        a.src = (A *)c->src;
        a.written = c->written;
        a.rec = (MoverRec<T> *)c->rec;
        a.nrec = c->nrec;
        a.flags = c->flags;
        a.spread = c->spread;
        a.inbox = c->inbox;
        a.deposit = deposit;
        a.p = c->prm;
        a.dt = (T)dt;
        for (int ax = 0; ax < 3; ++ax) {
            a.dt_h[ax] = (T)(dt / c->prm.h[ax]);
            a.g[ax] = (T)c->prm.g[ax];
        }
        a.tau_coef = (T)c->prm.tau_coef;
        for (int ax = 0; ax < 3; ++ax) a.g_dt[ax] = (T)(c->prm.g[ax] * dt);
        a.mass_coef = (T)c->prm.mass_coef;
        a.inv_V = (T)c->prm.inv_V;
        a.re2_coef = (T)(c->prm.re_coef * c->prm.re_coef);
        hipEvent_t ev[2] = {nullptr, nullptr};
        if (c->timing && deposit) {   // (not a step that the reverse recomputes)
            for (int k = 0; k < 2; ++k) {
                hipError_t ee = hipEventCreate(&ev[k]);
                if (ee != hipSuccess) return ee;
                c->tev.push_back(ev[k]);
            }
        }
        hipError_t r;
        switch (c->prm.E) {
        case 2: r = launch_step_e<T, A, 2>(c, a, s, ev); break;
        case 4: r = launch_step_e<T, A, 4>(c, a, s, ev); break;
        default: r = launch_step_e<T, A, 8>(c, a, s, ev); break;
        }
        if (r != hipSuccess) return r;

        return launch_rebin<T>(c, 0, s);
    });
}

hipError_t launch_flush_pending(st_ctx *c, hipStream_t s)
{
    hipLaunchKernelGGL(k_set_flag, dim3(1), dim3(1), 0, s, c->flags, (int)F_FORCE, 1);
    return dispatch(c, [&](auto t, auto) -> hipError_t {
        using T = decltype(t);
        return launch_rebin<T>(c, c->pending, s);
    });
}

hipError_t launch_stage_inject(st_ctx *c, int64_t n, const double *x, const double *up,
                               const double *d, int64_t at, hipStream_t s)
{
    return dispatch(c, [&](auto t, auto) -> hipError_t {
        using T = decltype(t);
        hipLaunchKernelGGL((k_stage<T>), dim3(grid_for(n)), dim3(256), 0, s, n, x, up, d, at,
                           c->next_id, c->prm, staging_of<T>(c), c->flags);
        return count_staged<T>(c, at, n, s);
    });
}

hipError_t launch_unstage(st_ctx *c, int64_t keep, hipStream_t s)
{
    const hipError_t e = launch_zero_i32(c->staged, c->C * c->staged_stride, s);
    if (e != hipSuccess) return e;
    return dispatch(c, [&](auto t, auto) -> hipError_t {
        return count_staged<decltype(t)>(c, 0, keep, s);
    });
}

// The two-pass read-out from this many particles on.  Droplets that lie evenly and
// are read again stay in the caches, where its two launches more cost some 8 us
// (binary32, 66 000 in 512 chunks: 21.5 us directly, 31 in two passes); where they
// have mixed or lie close together the direct one's scattered writes cost more
// (four plumes in 4096 chunks, 66 000: 40 and 25, 130 000: 65 and 40; one: 110 and
// 40, 212 and 89; in 32 768 chunks, evenly: 52 and 42).
constexpr int64_t kRecordsMin = 1 << 16;

hipError_t launch_get_particles(st_ctx *c, double *x, double *up, double *d, int64_t *id,
                                int32_t *cell, hipStream_t s)
{
    return dispatch(c, [&](auto t, auto) -> hipError_t {
        using T = decltype(t);
        const int64_t gi = c->max_items < 65536 ? c->max_items : 65536;
        const Store<T> st = store_of<T>(c);
        const ParticleOut out{x, up, d, id, cell};
        if (c->count < kRecordsMin || !second_store_free(c, s)) {
            hipLaunchKernelGGL((k_get_particles<T>), dim3(gi), dim3(256), 0, s, st, c->prm,
                               c->count, out);
            return hipGetLastError();
        }
        const dim3 g((c->count + 255) / 256);
        hipLaunchKernelGGL((k_records_clear<T>), g, dim3(256), 0, s, st, c->slots, c->count);
        hipLaunchKernelGGL((k_records_by_id<T>), dim3(gi), dim3(256), 0, s, st, c->slots,
                           c->count);
        hipLaunchKernelGGL((k_records_out<T>), g, dim3(256), 0, s, st, c->slots, c->prm, c->count,
                           out);
        return hipGetLastError();
    });
}

hipError_t launch_get_sources(st_ctx *c, double *out, int reset, hipStream_t s)
{
    return dispatch(c, [&](auto, auto acc) -> hipError_t {
        using A = decltype(acc);
        const Params &p = c->prm;
        const int32_t runs = (p.n[0] + kSrcCells - 1) / kSrcCells;
        const dim3 g(std::min<int64_t>((int64_t)runs * p.nc[1] * p.nc[2], 1 << 20));
        auto go = [&](auto k) {
            hipLaunchKernelGGL(k, g, dim3(256), 0, s, (A *)c->src, c->written, c->first[0],
                               c->first[1], c->flags, p, out, reset);
        };
        switch (p.E) {
        case 2: go(k_get_sources<A, 2>); break;
        case 4: go(k_get_sources<A, 4>); break;
        default: go(k_get_sources<A, 8>); break;
        }
        return hipGetLastError();
    });
}

// no chunk's sources hold anything
hipError_t launch_zero_sources(st_ctx *c, hipStream_t s)
{
    return launch_zero_i32(c->written, c->C, s);
}

hipError_t launch_zero_i32(int32_t *p, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n)), dim3(256), 0, s, p, n, 0);
    return hipGetLastError();
}

hipError_t launch_rotate_field(st_ctx *c, const void *u0, void *out, double cs, double sn,
                               hipStream_t s)
{
    return dispatch(c, [&](auto t, auto) -> hipError_t {
        using T = decltype(t);
        const int64_t ncell = (int64_t)c->prm.n[0] * c->prm.n[1] * c->prm.n[2];
        hipLaunchKernelGGL((k_rotate<T>), dim3(grid_for(ncell, 16384)), dim3(256), 0, s,
                           (const T *)u0, (T *)out, ncell, cs, sn);
        return hipGetLastError();
    });
}

// streaming reference: a plain copy with the particle state's access pattern
// (one 16-byte non-temporal load and store per thread)
typedef float f32x4 __attribute__((ext_vector_type(4)));
__global__ void __launch_bounds__(1024) k_stream_copy(const f32x4 *src, f32x4 *dst, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

hipError_t launch_stream_copy(const void *src, void *dst, int64_t bytes, hipStream_t s)
{
    const int64_t n = bytes / 16;
    int64_t g = (n + 1023) / 1024;
    if (g < 1) g = 1;
    if (g > (1 << 20)) g = 1 << 20;
    hipLaunchKernelGGL(k_stream_copy, dim3(g), dim3(1024), 0, s, (const f32x4 *)src,
                       (f32x4 *)dst, n);
    return hipGetLastError();
}

// extrapolator-corrector, elementwise over cells and components
__global__ void k_ec(int64_t n, int kind, const double *S_last, double *S_prev, double *E_prev,
                     double *applied)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double s = S_last[i];
        const double corrector = s - E_prev[i];
        double e = 0.0;
        if (kind == 1) e = s;
        if (kind == 2) e = 2.0 * s - S_prev[i];
        applied[i] = corrector + e;
        E_prev[i] = e;
        S_prev[i] = s;
    }
}

__global__ void k_zero_f64(double *p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.0;
}

hipError_t launch_ec(st_ctx *c, int kind, const double *S_last, double *applied, hipStream_t s)
{
    const int64_t n = 3 * (int64_t)c->prm.n[0] * c->prm.n[1] * c->prm.n[2];
    hipLaunchKernelGGL(k_ec, dim3(grid_for(n, 16384)), dim3(256), 0, s, n, kind, S_last,
                       c->ec_prev, c->ec_ext, applied);
    return hipGetLastError();
}

hipError_t launch_zero_f64(double *p, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero_f64, dim3(grid_for(n, 16384)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

size_t snapshot_bytes(const st_ctx *c)
{
    return snap_layout(c->slots, c->tsize, c->C, c->max_items).bytes;
}

// Saves the store (its arrivals placed first) and its containers into dst, or
// (restore) puts a saved store back.
hipError_t launch_snapshot(st_ctx *c, void *dst, int restore, hipStream_t s)
{
    const SnapLayout L = snap_layout(c->slots, c->tsize, c->C, c->max_items);
    if (!restore) {
        const hipError_t e = launch_settle(c, s);
        if (e != hipSuccess) return e;
    } else {
        wrote_store(c, s);
        hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(kSpreadInts)), dim3(256), 0, s, c->spread,
                           (int64_t)kSpreadInts, 0);
    }
    return dispatch(c, [&](auto t, auto) -> hipError_t {
        using T = decltype(t);
        hipLaunchKernelGGL((k_snapshot<T>), dim3(grid_for(c->slots, 16384)), dim3(256), 0, s,
                           views_of<T>(c), c->cont[0], c->cont[1], c->first[0], c->first[1],
                           c->slots, c->C, (char *)dst, L, c->flags, c->spread, restore);
        return hipGetLastError();
    });
}

}  // namespace st
