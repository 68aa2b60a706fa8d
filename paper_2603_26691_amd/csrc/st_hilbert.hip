// Placement of new particles by Hilbert-curve segments, and bounding boxes of
// particle partitions (paper Sec. 2.2, initialisation and chunk bounding
// boxes).
//
// Placement: the domain is a lattice of 2^order voxels per axis, visited in
// Hilbert-curve order and cut into nseg consecutive segments; segment s holds
// curve positions [floor(s V / nseg), floor((s+1) V / nseg)), V = 8^order.
// Particle k of a segment with nv voxels lies in its voxel floor(k nv / per_seg),
// at x_a = (c_a + u_a) (L_a / 2^order) for given uniforms u in [0, 1)^3: every
// segment holds exactly per_seg particles, voxel counts differ by at most one,
// and the particles follow the curve.  The mapping is global and
// deterministic, so any range of segments can be placed independently.
//
// Bounding boxes: partition p holds the particles with id in
// [id0 + p per_part, id0 + (p+1) per_part); its box is the componentwise
// minimum and maximum of their positions (positions as st_get_particles
// returns them).
#include "st_internal.h"

#include <algorithm>
#include <mutex>

// Partial results of st_bounding_boxes_noalloc (the min and max bounds of up
// to kNoAllocMaxParts boxes, as ordered integer images of binary64): a fixed
// device array, one copy per GPU, held until the process ends, so that the
// call allocates nothing.  Host code never passes this name to a kernel or a
// copy (on the host it is a stand-in, not a device address); it uses the
// per-device address that noalloc_scratch_init takes.
static __device__ __align__(256) unsigned long long scratch[st::kNoAllocMaxParts * 6];

namespace st {
namespace {

// bits 0, 3, 6, ... 27 of v, packed
__device__ __forceinline__ uint32_t every_third(uint32_t v)
{
    v &= 0x09249249u;
    v = (v | (v >> 2)) & 0x030C30C3u;
    v = (v | (v >> 4)) & 0x0300F00Fu;
    v = (v | (v >> 8)) & 0x030000FFu;
    return (v | (v >> 16)) & 0x3FFu;
}

// Hilbert curve position h (below 2^30) -> voxel: the index is split into its
// transpose (bit level l of axis i is bit 3 l + 2 - i of h), then Skilling's
// transpose-to-axes (AIP Conf. Proc. 707, 2004): Gray decode, then undo the
// reflections and exchanges from the least significant level up.
__device__ __forceinline__ void hilbert_voxel(int order, uint32_t h, uint32_t (&X)[3])
{
    X[0] = every_third(h >> 2);
    X[1] = every_third(h >> 1);
    X[2] = every_third(h);
    const uint32_t top = X[2] >> 1;
    X[2] ^= X[1];
    X[1] ^= X[0];
    X[0] ^= top;
    for (int l = 1; l < order; ++l) {
        const uint32_t P = (1u << l) - 1u;
#pragma unroll
        for (int i = 2; i >= 0; --i) {
            // all ones when the axis has bit l: the first axis is reflected,
            // else the low bits of the two axes are exchanged
            const uint32_t m = (uint32_t)-(int32_t)((X[i] >> l) & 1u);
            const uint32_t t = (X[0] ^ X[i]) & P & ~m;
            X[0] ^= (P & m) | t;
            if (i > 0) X[i] ^= t;
        }
    }
}

struct HilbertArgs {
    int32_t order;
    int64_t nseg, seg_begin, per_seg;
    int64_t q, r;        // V / nseg and V % nseg, V = 8^order voxels
    double hv[3];        // voxel width per axis, L / 2^order
};

// the first voxel of segment s: floor(s V / nseg) = s q + floor(s r / nseg)
template <class I>
__device__ __forceinline__ I segment_voxel(const HilbertArgs &a, I s)
{
    return s * (I)a.q + s * (I)a.r / (I)a.nseg;
}

// positions of particles first .. first + n - 1 of the call (particle g of the
// call is particle g mod per_seg of segment seg_begin + g / per_seg).  I: the
// integer type of the divisions; 32 bits where every product fits (a 64-bit
// division is a long sequence on this chip, and there are four a particle).
// The uniforms and positions pass through LDS, so that the lanes' accesses to
// the [n][3] arrays are consecutive.
// Bound by HBM (48 B a particle): 1e7 particles in 0.095 ms, 5.1 TB/s, against
// 0.135 ms with 64-bit divisions, bit-by-bit splitting and direct accesses.
template <class I>
__global__ void __launch_bounds__(256) k_hilbert_positions(HilbertArgs a, int64_t first,
                                                           int64_t n, const double *u, double *x)
{
    __shared__ double sh[3 * 256];
    for (int64_t b = (int64_t)blockIdx.x * 256; b < n; b += (int64_t)gridDim.x * 256) {
        const int nb = (int)(n - b < 256 ? n - b : 256);
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int e = threadIdx.x + 256 * j;
            if (e < 3 * nb) sh[e] = u[3 * b + e];
        }
        __syncthreads();
        if ((int)threadIdx.x < nb) {
            const I g = (I)(first + b + threadIdx.x);
            const I sl = g / (I)a.per_seg, k = g - sl * (I)a.per_seg;
            const I s = sl + (I)a.seg_begin;
            const I v0 = segment_voxel<I>(a, s), v1 = segment_voxel<I>(a, s + 1);
            const I v = v0 + k * (v1 - v0) / (I)a.per_seg;
            uint32_t c[3];
            hilbert_voxel(a.order, (uint32_t)v, c);
            for (int ax = 0; ax < 3; ++ax)
                sh[3 * threadIdx.x + ax] = ((double)c[ax] + sh[3 * threadIdx.x + ax]) * a.hv[ax];
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int e = threadIdx.x + 256 * j;
            if (e < 3 * nb) x[3 * b + e] = sh[e];
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// bounding boxes: positions are non-negative, so their binary64 bit patterns
// order like the values and the extrema are integer atomics on the patterns
// ---------------------------------------------------------------------------
constexpr unsigned long long kPosInf = 0x7FF0000000000000ull;
constexpr unsigned long long kNegInf = 0xFFF0000000000000ull;

__global__ void k_bbox_init(unsigned long long *box, int64_t nparts)
{
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < 6 * nparts;
         t += (int64_t)gridDim.x * blockDim.x)
        box[t] = (t % 6) < 3 ? kPosInf : 0ull;
}

// an empty partition keeps min = +inf; its max becomes -inf
__global__ void k_bbox_finish(unsigned long long *box, int64_t nparts)
{
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < nparts;
         p += (int64_t)gridDim.x * blockDim.x)
        if (box[6 * p] == kPosInf)
            for (int a = 0; a < 3; ++a) box[6 * p + 3 + a] = kNegInf;
}

__device__ __forceinline__ double wave_min(double v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ double wave_max(double v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    return v;
}

template <class T>
struct BoxArgs {
    Store<T> st;
    Params p;
    int64_t id0, per_part, nparts;
    unsigned long long *box;
};

// The partition (below nparts, else -1) and position of a slot of chunk cc.
template <class T>
__device__ __forceinline__ int64_t box_particle(const BoxArgs<T> &a, int32_t id, T x, T y, T z,
                                                T d, const int64_t (&cc)[3], double (&xg)[3])
{
    const Params &p = a.p;
    // a hole has the mark for an offset, or a negated diameter (binary64)
    if (!(x > T(kHoleMark) && d > T(0)) || id < a.id0) return -1;
    const int64_t rel = id - a.id0;    // below 2^31
    const int64_t part = a.per_part > 0x7fffffff ? 0 : (uint32_t)rel / (uint32_t)a.per_part;
    if (part >= a.nparts) return -1;
    const T o[3] = {x, y, z};
    for (int ax = 0; ax < 3; ++ax)   // binary32 metres in the FP32-everywhere form
        xg[ax] = p.global ? (double)o[ax] : ((double)(cc[ax] * p.E) + (double)o[ax]) * p.h[ax];
    return part;
}

// The tables lie in the re-bin's second store.
template <class T>
__device__ __forceinline__ unsigned long long *box_tables(const Store<T> &s)
{
    return reinterpret_cast<unsigned long long *>(s.V.pick(s.flags[F_CUR] ^ 1).ox);
}

// The boxes of up to kBoxTable partitions in LDS, workgroup by workgroup: a
// workgroup takes every gridDim.x-th container, four consecutive slots a
// thread, and keeps its own table of the partitions [blockIdx.y Kp,
// (blockIdx.y + 1) Kp).  A particle inside its partition's box as the table
// has it adds nothing (of n particles about ln n per bound do), so the atomics
// are few; the tables are then reduced over the workgroups.  Atomics on the
// boxes in memory are served beyond the XCD's own L2 (six a particle: 2.46 ms
// for 1e7 droplets in 4096 partitions, against 0.17 ms this way: 0.133 ms here,
// 0.037 ms the reduction).
constexpr int kBoxTable = 3328;      // 48 B each: 156 KB of the CU's 160 KB LDS
constexpr int kBoxPasses = 4;        // tables' worth of partitions (the store is read once each)
constexpr int kBoxGroups = 256;      // workgroups per table: one a CU

template <class T>
__global__ void __launch_bounds__(1024) k_bbox_tables(BoxArgs<T> a, int32_t Kp)
{
    extern __shared__ unsigned long long tab[];   // [Kp][6]
    constexpr int G = 16 / sizeof(T);
    typedef T vec __attribute__((ext_vector_type(G)));
    typedef int32_t ivec __attribute__((ext_vector_type(G)));
    static_assert(kAlign % G == 0, "container rooms must hold whole particle groups");
    const Params &p = a.p;
    const Current<T> S(a.st);
    const View<T> &V = S.V;
    const int32_t first = blockIdx.y * Kp;
    for (int t = threadIdx.x; t < 6 * Kp; t += 1024) tab[t] = (t % 6) < 3 ? kPosInf : 0ull;
    __syncthreads();
    auto take = [&](int64_t part, const double (&xg)[3]) {
        part -= first;
        if (part < 0 || part >= Kp) return;
        unsigned long long *b = tab + 6 * part;
        for (int ax = 0; ax < 3; ++ax) {
            const unsigned long long v = (unsigned long long)__double_as_longlong(xg[ax]);
            if (v < b[ax]) atomicMin(b + ax, v);
            if (v > b[3 + ax]) atomicMax(b + 3 + ax, v);
        }
    };
    for (int32_t it = blockIdx.x; it < S.ni; it += gridDim.x) {
        const ContState me = state_of(S.cont + it, S.m);
        const int64_t c = me.c;
        const int64_t cc[3] = {c % p.nc[0], (c / p.nc[0]) % p.nc[1],
                               c / ((int64_t)p.nc[0] * p.nc[1])};
        const int64_t s0 = me.base, s1 = s0 + me.cnt;
        // a group that runs past s1 stays inside the container's room
        for (int64_t q = s0 + G * (int64_t)threadIdx.x; q < s1; q += 1024 * G) {
            const vec x = *(const vec *)(V.ox + q), y = *(const vec *)(V.oy + q),
                      z = *(const vec *)(V.oz + q), d = *(const vec *)(V.d + q);
            const ivec id = *(const ivec *)(V.id + q);
#pragma unroll
            for (int k = 0; k < G; ++k) {
                double xg[3];
                if (q + k < s1)
                    take(box_particle<T>(a, id[k], x[k], y[k], z[k], d[k], cc, xg), xg);
            }
        }
        for (int32_t j = threadIdx.x; j < me.in; j += 1024) {
            const MoverRec<T> r = S.rec[me.ibase + j];
            double xg[3];
            take(box_particle<T>(a, r.id, r.ox, r.oy, r.oz, r.d, cc, xg), xg);
        }
    }
    __syncthreads();
    unsigned long long *out = box_tables(a.st) +
                              ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * 6 * Kp;
    for (int t = threadIdx.x; t < 6 * Kp; t += 1024) out[t] = tab[t];
}

// the tables of `groups` workgroups into the boxes
template <class T>
__global__ void __launch_bounds__(256) k_bbox_reduce(Store<T> st, int32_t groups, int32_t Kp,
                                                     int64_t nparts, unsigned long long *box)
{
    const unsigned long long *const tables = box_tables(st);
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= 6 * nparts) return;
    const int64_t part = t / 6, b = t - 6 * part;
    const int64_t pass = part / Kp;
    const unsigned long long *v = tables + (pass * groups * Kp + (part - pass * Kp)) * 6;
    unsigned long long lo = kPosInf, hi = 0ull;
#pragma unroll 8
    for (int32_t g = 0; g < groups; ++g) {
        const unsigned long long w = v[(int64_t)g * 6 * Kp + b];
        lo = w < lo ? w : lo;
        hi = w > hi ? w : hi;
    }
    // an empty partition keeps min = +inf; its max becomes -inf (positions are
    // non-negative, and 0.0 is the bit pattern 0, so its min tells)
    if (b >= 3) {
        unsigned long long m = kPosInf;
#pragma unroll 8
        for (int32_t g = 0; g < groups; ++g) {
            const unsigned long long w = v[(int64_t)g * 6 * Kp];
            m = w < m ? w : m;
        }
        if (m == kPosInf) hi = kNegInf;
    }
    box[t] = b < 3 ? lo : hi;
}

// One workgroup per container, updating the boxes in memory.  When every
// particle of a wave that belongs to a partition belongs to the same one (the
// usual case while partitions are compact), the wave reduces first and one
// lane updates the box.
template <class T>
__global__ void __launch_bounds__(256) k_bbox(BoxArgs<T> a)
{
    const Params &p = a.p;
    const Current<T> S(a.st);
    const View<T> &V = S.V;
    for (int32_t it = blockIdx.x; it < S.ni; it += gridDim.x) {
        const ContState me = state_of(S.cont + it, S.m);
        const int64_t c = me.c;
        const int64_t cc[3] = {c % p.nc[0], (c / p.nc[0]) % p.nc[1],
                               c / ((int64_t)p.nc[0] * p.nc[1])};
        const int32_t cnt = me.cnt, all = cnt + me.in;   // the arrivals last
        if (all == 0) continue;
        // A container's particles lie about in the order of their ids, so
        // workgroups that all began with the first would meet at the same boxes.
        const int32_t shift = (int32_t)((uint32_t)it * 2654435761u % (uint32_t)all);
        // every lane of the workgroup runs the same number of rounds
        for (int32_t o0 = 0; o0 < all; o0 += blockDim.x) {
            int32_t o = o0 + threadIdx.x;
            o = o < all ? (o + shift < all ? o + shift : o + shift - all) : all;
            int64_t part = -1;
            double xg[3] = {0.0, 0.0, 0.0};
            if (o < cnt) {
                const int64_t q = (int64_t)me.base + o;
                part = box_particle<T>(a, V.id[q], V.ox[q], V.oy[q], V.oz[q], V.d[q], cc, xg);
            } else if (o < all) {
                const MoverRec<T> r = S.rec[me.ibase + (o - cnt)];
                part = box_particle<T>(a, r.id, r.ox, r.oy, r.oz, r.d, cc, xg);
            }
            const uint64_t has = __ballot(part >= 0);
            if (has == 0) continue;
            const int lead = __ffsll((unsigned long long)has) - 1;
            const int64_t p0 = __shfl(part, lead);
            if (__ballot(part >= 0 && part != p0) == 0) {
                double lo[3], hi[3];
                for (int ax = 0; ax < 3; ++ax) {
                    lo[ax] = wave_min(part >= 0 ? xg[ax] : INFINITY);
                    hi[ax] = wave_max(part >= 0 ? xg[ax] : 0.0);
                }
                if (__lane_id() == lead)
                    for (int ax = 0; ax < 3; ++ax) {
                        atomicMin(a.box + 6 * p0 + ax, (unsigned long long)__double_as_longlong(lo[ax]));
                        atomicMax(a.box + 6 * p0 + 3 + ax,
                                  (unsigned long long)__double_as_longlong(hi[ax]));
                    }
            } else if (part >= 0) {
                for (int ax = 0; ax < 3; ++ax) {
                    const unsigned long long b = (unsigned long long)__double_as_longlong(xg[ax]);
                    atomicMin(a.box + 6 * part + ax, b);
                    atomicMax(a.box + 6 * part + 3 + ax, b);
                }
            }
        }
    }
}

inline int64_t blocks_for(int64_t n, int64_t cap = 8192)
{
    const int64_t b = (n + 255) / 256;
    return b < 1 ? 1 : (b > cap ? cap : b);
}

}  // namespace

hipError_t launch_hilbert_positions(int32_t order, int64_t nseg, int64_t seg_begin,
                                    int64_t per_seg, const double L[3], int64_t first, int64_t n,
                                    const double *u, double *x, hipStream_t s)
{
    HilbertArgs a;
    a.order = order;
    a.nseg = nseg;
    a.seg_begin = seg_begin;
    a.per_seg = per_seg;
    const int64_t V = (int64_t)1 << (3 * order);
    a.q = V / nseg;
    a.r = V % nseg;
    for (int ax = 0; ax < 3; ++ax) a.hv[ax] = L[ax] / (double)((int64_t)1 << order);
    const dim3 g(blocks_for(n, 1 << 20));
    // every product and index of the kernel below 2^32: s r with s <= nseg and
    // r < nseg, k (v1 - v0) with k < per_seg and v1 - v0 <= q + 1
    const int64_t lim = (int64_t)1 << 32;
    const bool narrow = first + n < lim && nseg < (1 << 16) && per_seg < lim / (a.q + 1);
    if (narrow)
        hipLaunchKernelGGL(k_hilbert_positions<uint32_t>, g, dim3(256), 0, s, a, first, n, u, x);
    else
        hipLaunchKernelGGL(k_hilbert_positions<int64_t>, g, dim3(256), 0, s, a, first, n, u, x);
    return hipGetLastError();
}

hipError_t launch_bounding_boxes(st_ctx *c, int64_t id0, int64_t per_part, int64_t nparts,
                                 double *box, hipStream_t s)
{
    unsigned long long *b = (unsigned long long *)box;
    // Tables when the partitions fit a few of them, the re-bin's second
    // store (second_store_free) has room for at least 32 workgroups' of them, and
    // their cost is less than what the direct updates may come to.  Beyond
    // kBoxPasses each further table reads the store again.
    //   The tables cost some 20 us and 1.5 us for each container that a workgroup
    // takes in turn (max_items / groups of them); direct updates cost more with
    // the particles, and with the particles that meet at one box where droplets
    // lie close together: 8000 in 57 partitions and 512 chunks, evenly spread 25 us
    // by tables and 33 directly, in one plume 25 and 175; 300 000 in 3000 and 32 768
    // chunks 2054 and 91.  Over 1206 calls of 300 to 300 000 droplets, 1 to 15 000
    // partitions and 0, 1 or 4 plumes this line takes 1.04 times what the better way
    // of each call does, always tables 1.43, always direct 2.26.
    const int64_t passes = (nparts + kBoxTable - 1) / kBoxTable;
    const int64_t Kp = (nparts + passes - 1) / passes;
    const int64_t room = c->slots * (int64_t)c->tsize / (passes * Kp * 48);
    const int64_t groups = std::min(std::min<int64_t>(kBoxGroups, room), c->max_items);
    const double worth = (double)c->count * (1.0 / 1500 + 1.0 / (16.0 * (double)nparts));
    const bool tables = worth * (double)groups >= (double)c->max_items &&
                        passes <= kBoxPasses && second_store_free(c, s) &&
                        groups >= std::min<int64_t>(32, c->max_items);
    auto run = [&](auto t) -> hipError_t {
        using T = decltype(t);
        BoxArgs<T> a{store_of<T>(c), c->prm, id0, per_part, nparts, b};
        if (tables) {
            hipError_t e = hipFuncSetAttribute((const void *)k_bbox_tables<T>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize,
                                               kBoxTable * 48);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL((k_bbox_tables<T>), dim3(groups, passes), dim3(1024),
                               (size_t)Kp * 48, s, a, (int32_t)Kp);
            hipLaunchKernelGGL((k_bbox_reduce<T>), dim3((6 * nparts + 255) / 256), dim3(256), 0, s,
                               a.st, (int32_t)groups, (int32_t)Kp, nparts, b);
            return hipGetLastError();
        }
        hipLaunchKernelGGL(k_bbox_init, dim3(blocks_for(6 * nparts)), dim3(256), 0, s, b, nparts);
        const int64_t gi = c->max_items < 65536 ? c->max_items : 65536;
        hipLaunchKernelGGL((k_bbox<T>), dim3(gi), dim3(256), 0, s, a);
        hipLaunchKernelGGL(k_bbox_finish, dim3(blocks_for(nparts)), dim3(256), 0, s, b, nparts);
        return hipGetLastError();
    };
    return c->form == ST_FORM_FP64 ? run(double(0)) : run(float(0));
}

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t noalloc_scratch_init(int device)
{
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[device]) return hipSuccess;
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[device] = static_cast<double *>(p);
    return hipSuccess;
}

hipError_t noalloc_scratch(int device, double **ptr)
{
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    *ptr = g_scratch_ptr[device];
    return *ptr ? hipSuccess : hipErrorNotInitialized;
}

}  // namespace st
