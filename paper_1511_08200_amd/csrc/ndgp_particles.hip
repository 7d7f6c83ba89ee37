// ndgp_particles.hip -- cloud-in-cell transfers between equal-mass particles
// and the grid levels (arXiv:1511.08200, Sec. IV.A: the density and the forces
// go back and forth between particles and cells by cloud-in-cell).
//
// A particle is a cube of one cell's size centred on its position: along each
// axis the cell whose centre lies below it gets 1 - t and the next one t (t:
// distance from that centre in cells), and a cell gets the product of its
// three axis weights.  Level 0 is the periodic domain; a patch level takes
// the particles whose cube overlaps its cells, comparing positions with the
// patch modulo the box (a patch may wrap the domain).
//
// Deposit: the weights are added as 64-bit fixed-point integers (2^-36 of a
// particle), so the sums are exact and the same in any order -- the density
// is bit for bit reproducible although thousands of threads add into one
// cell.  Gather: every particle reads the finest level whose eight cells
// around it all lie inside that level.

#include "ndgp_device.h"

#include <algorithm>
#include <cmath>

namespace ndgp {
namespace {

using namespace dev;

constexpr double kCicOne = 68719476736.0; // 2^36: one particle in fixed point

// w particles (0 <= w <= 1) in fixed point, rounded to nearest: adding 2^52 leaves
// the rounded integer in the low mantissa bits (w 2^36 is far below 2^52).  A weight
// that is no number (the position was none) is nothing: the maximum is 2^52 then.
__device__ __forceinline__ unsigned long long cic_fixed(double w) {
    const double r = fmax(fma(w, kCicOne, 0x1p52), 0x1p52);
    return (unsigned long long)__double_as_longlong(r) & 0xfffffffffffffull;
}

// distance from the level's lower corner along an axis, modulo the box, in
// domain cells: [0, n], n itself where the remainder of a tiny negative distance
// rounds up to it (its cells and weights are those of distance 0); n is a power of two,
// so 1 / n scales exactly
__device__ __forceinline__ double cic_distance(double x01, int n, double corner) {
    const double d = x01 * (double)n - corner;
    return d - (double)n * floor(d * (1.0 / (double)n));
}

// A level and, along one axis, the two neighbouring cells of a particle with
// their weights: `whole` if both lie in the level (always so on a periodic one).
// A patch may meet the particle or its image one box further down; where it
// spans the whole box, its last cell's upper neighbour is its first.  (Not the other
// way: a particle within half a cell above such a patch's lower corner has its lower
// cell at -1, and that weight is left out, as on any patch's edge.)
struct CicLevel {
    int n;               // domain cells per side
    double cx, cy, cz;   // the level's lower corner, domain cells
    double cells_per_domain;
    int m, periodic;
};
struct CicAxis {
    int i0, i1;
    double w0, w1;
    bool whole;
};

// KIND: the level is a patch, periodic, or (kCicEither) what L.periodic says
constexpr int kCicPatch = 0, kCicPeriodic = 1, kCicEither = 2;
template <int KIND>
__device__ __forceinline__ CicAxis cic_axis(const CicLevel &L, double x01, double corner) {
    const double d = cic_distance(x01, L.n, corner);
    const double u = d * L.cells_per_domain - 0.5, f = floor(u);
    CicAxis A;
    A.i0 = (int)f;
    A.w1 = u - f;
    A.w0 = 1.0 - A.w1;
    const int m = L.m;
    if (KIND == kCicPeriodic || (KIND == kCicEither && L.periodic)) {
        A.i1 = (A.i0 + 1) & (m - 1);
        A.i0 = A.i0 & (m - 1);
        A.whole = true;
        return A;
    }
    const double ub = (d - (double)L.n) * L.cells_per_domain - 0.5, fb = floor(ub);
    const int ib = (int)fb;
    const double tb = ub - fb;
    if ((unsigned)A.i0 < (unsigned)m) { // the particle itself, its upper cell perhaps the image's
        const bool up = A.i0 + 1 < m;
        A.i1 = up ? A.i0 + 1 : ib + 1;
        A.w1 = up ? A.w1 : tb;
        A.whole = up || (ib + 1 == 0 && A.i0 == m - 1);
    } else { // the image
        A.i0 = ib;
        A.i1 = ib + 1;
        A.w0 = 1.0 - tb;
        A.w1 = tb;
        A.whole = ib >= 0 && ib + 1 < m;
    }
    return A;
}

// candidate c of the four along an axis of a patch (bit 1: of the image, bit 0:
// the upper cell): its cell and weight; false outside the patch
__device__ __forceinline__ bool cic_candidate(const CicLevel &L, double d, int c, int &i,
                                              double &w) {
    const double u = (c & 2 ? d - (double)L.n : d) * L.cells_per_domain - 0.5, f = floor(u);
    const double t = u - f;
    i = (int)f + (c & 1);
    w = c & 1 ? t : 1.0 - t;
    return (unsigned)i < (unsigned)L.m;
}

// partial overlap with a patch (or no cell at all): straight to the accumulators
__device__ __forceinline__ void cic_add_partial(const CicLevel &L, double x, double y, double z,
                                                unsigned long long *__restrict__ acc) {
    const double dx = cic_distance(x, L.n, L.cx), dy = cic_distance(y, L.n, L.cy),
                 dz = cic_distance(z, L.n, L.cz);
    int i, j, k;
    double wx, wy, wz;
#pragma unroll 1
    for (int c = 0; c < 4; ++c) {
        if (!cic_candidate(L, dz, c, k, wz)) continue;
#pragma unroll 1
        for (int b = 0; b < 4; ++b) {
            if (!cic_candidate(L, dy, b, j, wy)) continue;
#pragma unroll 1
            for (int a = 0; a < 4; ++a) {
                if (!cic_candidate(L, dx, a, i, wx)) continue;
                const unsigned long long q = cic_fixed((wx * wy) * wz);
                if (q) atomicAdd(&acc[((size_t)k * L.m + j) * L.m + i], q);
            }
        }
    }
}

struct CicCloud {
    CicAxis x, y, z;
    bool whole;
};
template <int KIND>
__device__ __forceinline__ CicCloud cic_cloud(const CicLevel &L, double x, double y, double z) {
    CicCloud c;
    c.x = cic_axis<KIND>(L, x, L.cx);
    c.y = cic_axis<KIND>(L, y, L.cy);
    c.z = cic_axis<KIND>(L, z, L.cz);
    c.whole = c.x.whole && c.y.whole && c.z.whole;
    return c;
}

// the eight weights of a whole particle, in fixed point
__device__ __forceinline__ void cic_weights(const CicCloud &cl, unsigned long long q[8]) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int a = 0; a < 2; ++a)
                q[(c * 2 + b) * 2 + a] =
                    cl.whole ? cic_fixed(((a ? cl.x.w1 : cl.x.w0) * (b ? cl.y.w1 : cl.y.w0)) *
                                         (c ? cl.z.w1 : cl.z.w0))
                             : 0ull;
}

// Lanes of a wave that hold a contiguous run of equal keys add their weights
// (a segmented scan by shuffles); true on the lane that ends up with the run's
// sum, its last.
__device__ __forceinline__ bool cic_merge_runs(long long key, unsigned long long q[8]) {
    const int lane = threadIdx.x & 63;
    const long long kprev = __shfl_up(key, 1, 64);
    const bool head = lane == 0 || kprev != key;
    // start lane of this lane's run of equal keys (max over heads at or below)
    int seg = head ? lane : 0;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(seg, off, 64);
        if (lane >= off) seg = seg > o ? seg : o;
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int so = __shfl_up(seg, off, 64);
        unsigned long long qo[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) qo[r] = __shfl_up(q[r], off, 64);
        if (lane >= off && so == seg) {
#pragma unroll
            for (int r = 0; r < 8; ++r) q[r] += qo[r];
        }
    }
    const int snext = __shfl_down(seg, 1, 64);
    return lane == 63 || snext != seg;
}

// One thread per particle, straight into the accumulators.  Particles whose
// eight cells are all in the level (the usual case) are keyed by their lower
// cell; lanes of a wave that hold a contiguous run of equal keys -- particles
// sorted by cell, as a tree code keeps them, in a dense region -- first add
// their fixed-point weights, and only the run's last lane sends the eight
// atomics.  Integer sums: the same bits whatever the grouping.  Bound by those
// device-scope atomics, which complete at the memory side (the L2s of the eight
// XCDs are not coherent with each other): 22 G/s, 5.8 ms for 256^3 particles in
// no spatial order on 256^3 cells.
__global__ void __launch_bounds__(kBlock)
k_cic_deposit(const double *__restrict__ pos, long long np, CicLevel L,
              unsigned long long *__restrict__ acc) {
    const long long p = (long long)blockIdx.x * kBlock + threadIdx.x;
    const int lane = threadIdx.x & 63;
    CicCloud cl;
    cl.whole = false;
    if (p < np) {
        const double x = pos[p], y = pos[np + p], z = pos[2 * np + p];
        cl = cic_cloud<kCicEither>(L, x, y, z);
        if (!cl.whole) cic_add_partial(L, x, y, z, acc);
    }
    unsigned long long q[8];
    cic_weights(cl, q);
    // key: lower cell of a whole particle, else unique to the lane
    const long long key =
        cl.whole ? (long long)(((size_t)cl.z.i0 * L.m + cl.y.i0) * L.m + cl.x.i0) : -1 - lane;
    const bool tail = cic_merge_runs(key, q);
    if (cl.whole && tail) {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    const unsigned long long v = q[(c * 2 + b) * 2 + a];
                    const int i = a ? cl.x.i1 : cl.x.i0, j = b ? cl.y.i1 : cl.y.i0,
                              k = c ? cl.z.i1 : cl.z.i0;
                    if (v) atomicAdd(&acc[((size_t)k * L.m + j) * L.m + i], v);
                }
    }
}

// ---- the binned deposit ----------------------------------------------------
//
// Particles sorted by tile add their weights in LDS, so that the memory side
// sees one value per cell and tile instead of eight atomics per particle.  A
// tile is 2^LX x 2^LY x 2^LZ cells; it owns the particles whose lower cell it
// holds, and its LDS block has one more cell per axis for their upper cells.
//   k_cic_count    counts each workgroup's particles per tile (LDS) and takes
//                  the workgroup's place in every tile's list
//   k_cic_scan     first particle of every tile; cuts long lists into segments
//   k_cic_scatter  writes x, y, z of every particle to its place
//   k_cic_tiles    one workgroup per segment: LDS sums, then the tile's cells
// Cells strictly inside a tile are written by its one workgroup alone; the
// faces, and the tiles with several segments, add by atomics.  The sums are
// integers, so the result is bit for bit that of k_cic_deposit.
// 256^3 particles in no order on 256^3 cells, us: count 121 and scatter 381 (the
// positions read twice and written once; the scattered 24-byte writes leave L2
// partly filled), tiles 278 (positions and cells at 1.9 TB/s, beside 134 M LDS
// atomics), clearing and converting the accumulators 71: 0.86 ms, against 5.9 ms
// of k_cic_deposit.

constexpr int kCicSortThreads = 1024;

template <int LX, int LY, int LZ>
__device__ __forceinline__ int cic_bin(const CicLevel &L, const CicCloud &c) {
    const int nbx = L.m >> LX, nby = L.m >> LY;
    return ((c.z.i0 >> LZ) * nby + (c.y.i0 >> LY)) * nbx + (c.x.i0 >> LX);
}

// add one per lane with bin >= 0 to cnt[bin] and return the counter's value
// before it; a wave whose lanes share one tile (sorted particles) sends one atomic
__device__ __forceinline__ unsigned cic_take(unsigned *cnt, int bin) {
    const int first = __builtin_amdgcn_readfirstlane(bin);
    const unsigned long long same = __ballot(bin == first);
    if (first >= 0 && same == __ballot(true)) {
        const int lane = threadIdx.x & 63;
        const unsigned long long below = same & ((1ull << lane) - 1);
        unsigned v = 0;
        if (below == 0) v = atomicAdd(&cnt[first], (unsigned)__popcll(same));
        v = __shfl(v, __ffsll(same) - 1, 64);
        return v + (unsigned)__popcll(below);
    }
    return bin >= 0 ? atomicAdd(&cnt[bin], 1u) : 0u;
}

// A thread's particles are taken kCicBatch at a time, all their loads first.
constexpr int kCicBatch = 4;

template <int KIND, int LX, int LY, int LZ>
__global__ void __launch_bounds__(kCicSortThreads)
k_cic_count(const double *__restrict__ pos, long long np, long long first, unsigned count,
            int per_thread, CicLevel L, int bins, unsigned *__restrict__ counts,
            unsigned *__restrict__ table, unsigned long long *__restrict__ acc) {
    extern __shared__ unsigned local[];
    for (int b = threadIdx.x; b < bins; b += kCicSortThreads) local[b] = 0u;
    __syncthreads();
    for (int e0 = 0; e0 < per_thread; e0 += kCicBatch) {
        double x[kCicBatch], y[kCicBatch], z[kCicBatch];
        bool on[kCicBatch];
#pragma unroll
        for (int e = 0; e < kCicBatch; ++e) {
            const unsigned i =
                (blockIdx.x * (unsigned)per_thread + e0 + e) * kCicSortThreads + threadIdx.x;
            on[e] = e0 + e < per_thread && i < count;
            const long long p = first + (on[e] ? i : 0u);
            x[e] = pos[p];
            y[e] = pos[np + p];
            z[e] = pos[2 * np + p];
        }
#pragma unroll
        for (int e = 0; e < kCicBatch; ++e) {
            const CicCloud cl = cic_cloud<KIND>(L, x[e], y[e], z[e]);
            int bin = -1;
            if (on[e] && cl.whole) bin = cic_bin<LX, LY, LZ>(L, cl);
            if constexpr (KIND == kCicPatch)
                if (on[e] && !cl.whole) cic_add_partial(L, x[e], y[e], z[e], acc);
            cic_take(local, bin);
        }
    }
    __syncthreads();
    for (int b = threadIdx.x; b < bins; b += kCicSortThreads)
        if (local[b]) table[(size_t)blockIdx.x * bins + b] = atomicAdd(&counts[b], local[b]);
}

// one workgroup: exclusive sums of the tile counts and of their segments of at
// most `seg` particles; clears the counts for the next chunk
__global__ void __launch_bounds__(kCicSortThreads)
k_cic_scan(unsigned *__restrict__ counts, int bins, unsigned seg, unsigned *__restrict__ base,
           CicSegment *__restrict__ segments, unsigned *__restrict__ n_segments) {
    __shared__ unsigned wp[kCicSortThreads / 64], wg[kCicSortThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int each = (bins + kCicSortThreads - 1) / kCicSortThreads;
    unsigned np = 0, ng = 0;
    for (int e = 0; e < each; ++e) {
        const int b = tid * each + e;
        if (b < bins) {
            np += counts[b];
            ng += (counts[b] + seg - 1) / seg;
        }
    }
    unsigned p = np, g = ng; // inclusive sums over the wave, then over the waves
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned po = __shfl_up(p, off, 64), go = __shfl_up(g, off, 64);
        if (lane >= off) {
            p += po;
            g += go;
        }
    }
    if (lane == 63) {
        wp[wave] = p;
        wg[wave] = g;
    }
    __syncthreads();
    for (int w = 0; w < wave; ++w) {
        p += wp[w];
        g += wg[w];
    }
    if (tid == kCicSortThreads - 1) *n_segments = g;
    p -= np;
    g -= ng;
    for (int e = 0; e < each; ++e) {
        const int b = tid * each + e;
        if (b >= bins) break;
        const unsigned c = counts[b];
        counts[b] = 0u;
        base[b] = p;
        for (unsigned o = 0; o < c; o += seg, ++g)
            segments[g] = CicSegment{(unsigned)b, p + o, c - o < seg ? c - o : seg, c <= seg ? 1u : 0u};
        p += c;
    }
}

template <int KIND, int LX, int LY, int LZ>
__global__ void __launch_bounds__(kCicSortThreads)
k_cic_scatter(const double *__restrict__ pos, long long np, long long first, unsigned count,
              int per_thread, CicLevel L, int bins, const unsigned *__restrict__ base,
              const unsigned *__restrict__ table, double *__restrict__ sorted) {
    extern __shared__ unsigned local[];
    for (int b = threadIdx.x; b < bins; b += kCicSortThreads) // entries of empty tiles: not used
        local[b] = base[b] + table[(size_t)blockIdx.x * bins + b];
    __syncthreads();
    for (int e0 = 0; e0 < per_thread; e0 += kCicBatch) {
        double x[kCicBatch], y[kCicBatch], z[kCicBatch];
        bool on[kCicBatch];
#pragma unroll
        for (int e = 0; e < kCicBatch; ++e) {
            const unsigned i =
                (blockIdx.x * (unsigned)per_thread + e0 + e) * kCicSortThreads + threadIdx.x;
            on[e] = e0 + e < per_thread && i < count;
            const long long p = first + (on[e] ? i : 0u);
            x[e] = pos[p];
            y[e] = pos[np + p];
            z[e] = pos[2 * np + p];
        }
#pragma unroll
        for (int e = 0; e < kCicBatch; ++e) {
            const CicCloud cl = cic_cloud<KIND>(L, x[e], y[e], z[e]);
            const int bin = on[e] && cl.whole ? cic_bin<LX, LY, LZ>(L, cl) : -1;
            const unsigned at = cic_take(local, bin);
            if (bin >= 0) {
                double *o = sorted + 3 * (size_t)at;
                o[0] = x[e];
                o[1] = y[e];
                o[2] = z[e];
            }
        }
    }
}

template <int KIND, int LX, int LY, int LZ, int NT>
__global__ void __launch_bounds__(NT)
k_cic_tiles(const double *__restrict__ sorted, const CicSegment *__restrict__ segments,
            const unsigned *__restrict__ n_segments, CicLevel L, int fresh_acc,
            unsigned long long *__restrict__ acc) {
    constexpr int PX = (1 << LX) + 1, PY = (1 << LY) + 1, PZ = (1 << LZ) + 1;
    __shared__ unsigned long long T[PX * PY * PZ];
    if (blockIdx.x >= *n_segments) return;
    const CicSegment sg = segments[blockIdx.x];
    const int nbx = L.m >> LX, nby = L.m >> LY;
    const int x0 = ((int)sg.bin % nbx) << LX, y0 = ((int)sg.bin / nbx % nby) << LY,
              z0 = ((int)sg.bin / (nbx * nby)) << LZ;
    for (int q = threadIdx.x; q < PX * PY * PZ; q += NT) T[q] = 0ull;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const double *mine = sorted + 3 * (size_t)sg.first;
    for (unsigned i0 = threadIdx.x; i0 < sg.count + threadIdx.x; i0 += kCicBatch * NT) {
        double x[kCicBatch], y[kCicBatch], z[kCicBatch];
#pragma unroll
        for (int e = 0; e < kCicBatch; ++e) {
            const unsigned i = i0 + e * NT < sg.count ? i0 + e * NT : 0u;
            x[e] = mine[3 * (size_t)i];
            y[e] = mine[3 * (size_t)i + 1];
            z[e] = mine[3 * (size_t)i + 2];
        }
#pragma unroll
        for (int e = 0; e < kCicBatch; ++e) {
            CicCloud cl = cic_cloud<KIND>(L, x[e], y[e], z[e]);
            cl.whole = i0 + e * NT < sg.count; // only whole particles were sorted
            const int at = ((cl.z.i0 - z0) * PY + cl.y.i0 - y0) * PX + cl.x.i0 - x0;
            unsigned long long q[8];
            cic_weights(cl, q);
            // sorted particles of a dense region: runs of one cell are added up first
            const int key = cl.whole ? at : -1 - lane, kprev = __shfl_up(key, 1, 64);
            bool add = cl.whole;
            if (__popcll(__ballot(lane == 0 || kprev != key)) <= 16)
                add = cic_merge_runs(key, q) && cl.whole;
            if (add) {
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int a = 0; a < 2; ++a)
                            atomicAdd(&T[at + (c * PY + b) * PX + a], q[(c * 2 + b) * 2 + a]);
            }
        }
    }
    __syncthreads();
    const int msk = L.m - 1;
    for (int q = threadIdx.x; q < PX * PY * PZ; q += NT) {
        const unsigned long long v = T[q];
        const int lx = q % PX, ly = q / PX % PY, lz = q / (PX * PY);
        const int x = (x0 + lx) & msk, y = (y0 + ly) & msk, z = (z0 + lz) & msk;
        unsigned long long *dst = acc + ((size_t)z * L.m + y) * L.m + x;
        const bool inner = lx > 0 && lx < PX - 1 && ly > 0 && ly < PY - 1 && lz > 0 && lz < PZ - 1;
        if (inner && sg.whole) { // no other workgroup adds here
            if (fresh_acc) *dst = v;
            else if (v) *dst += v;
        } else if (v) {
            atomicAdd(dst, v);
        }
    }
}

__global__ void __launch_bounds__(kBlock)
k_cic_finish(const unsigned long long *__restrict__ acc, size_t cells, double scale,
             double *__restrict__ delta) {
    const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (t < cells) delta[t] = (double)acc[t] * scale - 1.0;
}

__global__ void __launch_bounds__(kBlock)
k_zero_acc(unsigned long long *__restrict__ a, size_t count) {
    const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (t < count) a[t] = 0ull;
}

// The lower cell and weight along one axis if all of the particle's cells lie
// inside the level (for a patch: the image whose two cells are in [0, m)).
__device__ __forceinline__ bool cic_inside(double x01, int n, double corner,
                                           double cells_per_domain, int m, bool periodic,
                                           int &i0, double &t) {
    const double d = cic_distance(x01, n, corner);
#pragma unroll
    for (int img = 0; img < 2; ++img) {
        if (periodic && img) break;
        const double u = (img ? d - (double)n : d) * cells_per_domain - 0.5;
        const double f = floor(u);
        const int i = (int)f;
        if (periodic || (i >= 0 && i + 1 <= m - 1)) {
            i0 = i;
            t = u - f;
            return true;
        }
    }
    return false;
}

// Gather.  Bound by the cache lines it touches: for particles in no order the two
// x-neighbours of a row lie in one 128-byte line of each component, so twelve lines
// per particle, which the fabric delivers at 6 TB/s (9 TB/s where the three
// components fit the 256 MB memory-side cache).
//
// k_cic_gather_parts: one component per block, the blocks of the first component
// first.  The lines in flight then belong to one array, a third of the footprint, and
// a thread holds a third of the sums; the positions are read three times.
//
// With a workspace (`lines`) the domain's components may be interleaved first, x y z
// of a cell together: five lines instead of twelve, for one more pass over the cells,
// and k_cic_gather_cells takes the three sums of a particle in one thread.  With more
// particles than cells that is the faster for particles in any order; with fewer, not
// for those in cell order, which touch few lines anyway: there a sample of neighbouring
// particles decides on the device (*lines_off), and one of the two kernels returns at
// once.  The arithmetic is the same everywhere.
//
// 2^24 particles, us a call: one thread per particle on component arrays / one
// component per block / interleaved
//   no order    32^3 1560 / 926 / 562, 64^3 2130 / 1006 / 892, 128^3 3750 / 2930 / 1533,
//               256^3 4270 / 3950 / 1837, 512^3 5440 / 4350 / 3500
//   cell order  32^3 446 / 551 / 356, 128^3 443 / 556 / 387, 256^3 634 / 577 / 591,
//               512^3 1490 / 1068 / 1950
// Two cells per thread: 48 bytes in a row written (cells is a power of two, lines
// 16-byte aligned).  ASK: not for particles in cell order, which every block finds out
// from the same kBlock pairs of neighbouring particles (a launch less than asking
// first), and the first one leaves in *lines_off.
template <bool ASK>
__global__ void __launch_bounds__(kBlock)
k_cic_interleave(const double *__restrict__ f, size_t cells, double *__restrict__ lines,
                 const double *__restrict__ pos, long long np, int n,
                 unsigned *__restrict__ lines_off) {
    if constexpr (ASK) {
        const long long p = (np - 1) * (int)threadIdx.x / kBlock; // and p + 1 < np
        const double reach[3] = {16.0, 2.0, 2.0};                 // cells in x, y, z
        bool near = true;
#pragma unroll
        for (int a = 0; a < 3; ++a)
            near = near && fabs(pos[a * np + p + 1] - pos[a * np + p]) * n <= reach[a];
        const bool off = 2 * __syncthreads_count(near) > kBlock;
        if (blockIdx.x == 0 && threadIdx.x == 0) *lines_off = off ? 1u : 0u;
        if (off) return;
    }
    for (size_t c = 2 * ((size_t)blockIdx.x * kBlock + threadIdx.x); c < cells;
         c += 2 * (size_t)gridDim.x * kBlock) {
        double v[6];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            v[a] = f[a * cells + c];
            v[3 + a] = f[a * cells + c + 1];
        }
        double2 *o = reinterpret_cast<double2 *>(lines + 3 * c);
        o[0] = make_double2(v[0], v[1]);
        o[1] = make_double2(v[2], v[3]);
        o[2] = make_double2(v[4], v[5]);
    }
}

// PARTS components at a particle from the cells of a level: STRIDE values from
// cell to cell, `pitch` from component to component
template <int PARTS, int STRIDE>
__device__ __forceinline__ void cic_gather_cells(const double *f, size_t pitch, int m, bool per,
                                                 int i0, int j0, int k0, double tx, double ty,
                                                 double tz, double acc[PARTS]) {
#pragma unroll
    for (int a = 0; a < PARTS; ++a) acc[a] = 0.0;
#pragma unroll
    for (int dz = 0; dz < 2; ++dz)
#pragma unroll
        for (int dy = 0; dy < 2; ++dy)
#pragma unroll
            for (int dx = 0; dx < 2; ++dx) {
                const double w =
                    ((dx ? tx : 1.0 - tx) * (dy ? ty : 1.0 - ty)) * (dz ? tz : 1.0 - tz);
                int ci = i0 + dx, cj = j0 + dy, ck = k0 + dz;
                if (per) {
                    ci &= m - 1;
                    cj &= m - 1;
                    ck &= m - 1;
                }
                const double *v = f + STRIDE * (((size_t)ck * m + cj) * m + ci);
#pragma unroll
                for (int a = 0; a < PARTS; ++a) acc[a] = fma(w, v[a * pitch], acc[a]);
            }
}

// the finest level whose eight cells around the particle all lie inside it, their
// lower cell and the weights
__device__ __forceinline__ int cic_finest(const CicLevels &lv, double x, double y, double z,
                                          int &i0, int &j0, int &k0, double &tx, double &ty,
                                          double &tz) {
    for (int q = lv.levels - 1; q > 0; --q) {
        const int m = lv.m[q];
        const double cpd = lv.cells_per_domain[q];
        if (cic_inside(x, lv.n, lv.corner[q][0], cpd, m, false, i0, tx) &&
            cic_inside(y, lv.n, lv.corner[q][1], cpd, m, false, j0, ty) &&
            cic_inside(z, lv.n, lv.corner[q][2], cpd, m, false, k0, tz))
            return q;
    }
    cic_inside(x, lv.n, lv.corner[0][0], 1.0, lv.n, true, i0, tx);
    cic_inside(y, lv.n, lv.corner[0][1], 1.0, lv.n, true, j0, ty);
    cic_inside(z, lv.n, lv.corner[0][2], 1.0, lv.n, true, k0, tz);
    return 0;
}

// with lines_off: only if it is set
__global__ void __launch_bounds__(kBlock)
k_cic_gather_parts(const double *__restrict__ pos, long long np, unsigned blocks, CicLevels lv,
                   const unsigned *__restrict__ lines_off, double *__restrict__ out) {
    if (lines_off && !*lines_off) return;
    for (unsigned b = blockIdx.x; b < 3 * blocks; b += gridDim.x) {
        const int part = b / blocks;
        const long long p = (long long)(b - part * blocks) * kBlock + threadIdx.x;
        if (p >= np) continue;
        int i0, j0, k0;
        double tx, ty, tz, acc[1];
        const int q = cic_finest(lv, pos[p], pos[np + p], pos[2 * np + p], i0, j0, k0, tx, ty, tz);
        const int m = lv.m[q];
        cic_gather_cells<1, 1>(lv.force[q] + part * ((size_t)m * m * m), 0, m, q == 0, i0, j0, k0,
                               tx, ty, tz, acc);
        out[part * np + p] = acc[0];
    }
}

// lines: the domain's components interleaved (null: they are not); with lines_off: only
// if it is not set.  A particle's position is read before its sums are written, by the
// same thread: `out` may be `pos`.
__global__ void __launch_bounds__(kBlock)
k_cic_gather_cells(const double *pos, long long np, unsigned blocks, CicLevels lv,
                   const double *__restrict__ lines, const unsigned *__restrict__ lines_off,
                   double *out) {
    if (lines_off && *lines_off) return;
    for (unsigned b = blockIdx.x; b < blocks; b += gridDim.x) {
        const long long p = (long long)b * kBlock + threadIdx.x;
        if (p >= np) continue;
        int i0, j0, k0;
        double tx, ty, tz, acc[3];
        const int q = cic_finest(lv, pos[p], pos[np + p], pos[2 * np + p], i0, j0, k0, tx, ty, tz);
        const int m = lv.m[q];
        if (lines && q == 0)
            cic_gather_cells<3, 3>(lines, 1, m, true, i0, j0, k0, tx, ty, tz, acc);
        else
            cic_gather_cells<3, 1>(lv.force[q], (size_t)m * m * m, m, q == 0, i0, j0, k0, tx, ty,
                                   tz, acc);
#pragma unroll
        for (int a = 0; a < 3; ++a) out[a * np + p] = acc[a];
    }
}

// Refinement criterion of Sec. IV.A: a cell is refined when the particles in
// its volume number more than n_ref.  count = (delta + 1) mean with mean the
// level's particles per cell; per-block counts of flagged cells.
__global__ void __launch_bounds__(kBlock)
k_refine_flags(const double *__restrict__ delta, size_t cells, double mean, double n_ref,
               unsigned char *__restrict__ flags, double *__restrict__ partials) {
    double nflag = 0.0;
    for (size_t c = (size_t)blockIdx.x * kBlock + threadIdx.x; c < cells;
         c += (size_t)gridDim.x * kBlock) {
        const bool f = (delta[c] + 1.0) * mean > n_ref;
        flags[c] = f ? 1 : 0;
        nflag += f ? 1.0 : 0.0;
    }
    const double b = block_sum(nflag);
    if (threadIdx.x == 0) partials[blockIdx.x] = b;
}

} // namespace

void launch_refine_flags(const double *delta, size_t cells, double mean, double n_ref,
                         unsigned char *flags, double *partials, hipStream_t st) {
    k_refine_flags<<<kReduceBlocks, kBlock, 0, st>>>(delta, cells, mean, n_ref, flags, partials);
}

// Tiles by level size: small enough for a few hundred of them on a small level
// (8^3 cells), and as large as LDS holds on the largest (32 x 32 x 16: 148 KB),
// where a workgroup's sort writes longer runs per tile and fewer cells lie on
// faces.  1024^3 levels (65536 tiles) are not binned: their counters exceed LDS.
// A segment has some four particles per cell of the LDS block at least, so that
// writing the block costs a small part of the atomics it saves.
struct CicTiling {
    int lx, ly, lz;
    unsigned seg;
};
static CicTiling cic_tiling(int m) {
    if (m <= 64) return {3, 3, 3, 4096};
    if (m <= 128) return {4, 4, 4, 16384};
    return {5, 5, 4, 65536};
}

int cic_bins(int m) {
    if (m > 512) return 0;
    const CicTiling t = cic_tiling(m);
    return (m >> t.lx) * (m >> t.ly) * (m >> t.lz);
}

size_t cic_segments(int m, size_t chunk) {
    return cic_bins(m) ? (size_t)cic_bins(m) + chunk / cic_tiling(m).seg : 0;
}

size_t cic_chunk(int n) {
    const size_t cells = (size_t)n * n * n;
    return cells < ((size_t)1 << 20) ? (size_t)1 << 20
                                     : cells > ((size_t)1 << 24) ? (size_t)1 << 24 : cells;
}

size_t cic_acc_words(int m) {
    return (size_t)m * m * m + ((size_t)cic_bins(m) + 1) / 2; // then one 32-bit counter per tile
}

// From how many particles on sorting a level pays: below, its extra launches and the
// tiles it writes cost more than the atomics it saves.  Measured (particles in no order,
// on a domain; direct / binned, us): 32^3 cells 35 / 39 at 32768 and 58 / 31 at 65536;
// 128^3 42 / 47 at 65536 and 67 / 50 at 131072; 256^3 113 / 140 at 131072, 159 / 147 at
// 262144 and 5856 / 855 at 2^24; 512^3 960 / 1183 at 2^20 and 2079 / 1459 at 2^22.
//
// On a refinement it saves what the particles inside cost, which is not known before
// they have been looked at: 20 us at 32^3 and 64^3 cells, 30 at 128^3 and 85 at 256^3
// go, whether few of them meet it (64^3 in 256^3, 300000 in no order: 228 us for both
// levels instead of 208) or most of a dense field (32^3 in 64^3, as many: 112 instead
// of 216).  So a refinement is sorted from the sum of all levels' lines on: what its
// sort may cost is then saved already on the levels above (0.3 ns per particle beyond
// their lines).
static long long cic_sort_line(int m) {
    return 49152 + (long long)((size_t)m * m * m / 64);
}

void cic_sorted_levels(const int *m, int levels, long long np, bool *sorted) {
    long long all = 0;
    for (int l = 0; l < levels; ++l) all += cic_sort_line(m[l]);
    for (int l = 0; l < levels; ++l)
        sorted[l] = cic_bins(m[l]) > 0 && np >= (l == 0 ? cic_sort_line(m[0]) : all);
}

void launch_zero_words(unsigned long long *a, size_t count, hipStream_t st) {
    k_zero_acc<<<blocks_for(count), kBlock, 0, st>>>(a, count);
}

template <int KIND, int LX, int LY, int LZ, int NT>
static void cic_binned(const double *pos, long long np, const CicLevel &L, unsigned seg,
                       unsigned long long *acc, const CicScratch &scr, hipStream_t st) {
    const int bins = cic_bins(L.m);
    unsigned *counts = reinterpret_cast<unsigned *>(acc + (size_t)L.m * L.m * L.m);
    for (long long first = 0; first < np; first += (long long)scr.chunk) {
        const unsigned count =
            (unsigned)(np - first < (long long)scr.chunk ? np - first : (long long)scr.chunk);
        const unsigned per_block = (count + kCicBlocks - 1) / kCicBlocks;
        const int per_thread = (int)((per_block + kCicSortThreads - 1) / kCicSortThreads);
        const unsigned blocks =
            (count + per_thread * kCicSortThreads - 1) / (per_thread * kCicSortThreads);
        const size_t lds = (size_t)bins * sizeof(unsigned);
        k_cic_count<KIND, LX, LY, LZ><<<blocks, kCicSortThreads, lds, st>>>(
            pos, np, first, count, per_thread, L, bins, counts, scr.table, acc);
        k_cic_scan<<<1, kCicSortThreads, 0, st>>>(counts, bins, seg, scr.base, scr.segments,
                                                  scr.n_segments);
        k_cic_scatter<KIND, LX, LY, LZ><<<blocks, kCicSortThreads, lds, st>>>(
            pos, np, first, count, per_thread, L, bins, scr.base, scr.table, scr.sorted);
        k_cic_tiles<KIND, LX, LY, LZ, NT><<<(unsigned)((size_t)bins + count / seg), NT, 0, st>>>(
            scr.sorted, scr.segments, scr.n_segments, L, KIND == kCicPeriodic && first == 0 ? 1 : 0, acc);
    }
}

template <int KIND>
static void cic_binned(const double *pos, long long np, const CicLevel &L,
                       unsigned long long *acc, const CicScratch &scr, hipStream_t st) {
    const CicTiling t = cic_tiling(L.m);
    if (t.lx == 3)
        cic_binned<KIND, 3, 3, 3, 256>(pos, np, L, t.seg, acc, scr, st);
    else if (t.lx == 4)
        cic_binned<KIND, 4, 4, 4, 512>(pos, np, L, t.seg, acc, scr, st);
    else
        cic_binned<KIND, 5, 5, 4, 1024>(pos, np, L, t.seg, acc, scr, st);
}

void launch_cic_deposit(const double *pos, long long np, int n, const double corner[3], int q,
                        int m, unsigned long long *acc, double *delta, const CicScratch &scr,
                        hipStream_t st) {
    const size_t cells = (size_t)m * m * m;
    const CicLevel L{n, corner[0], corner[1], corner[2], std::ldexp(1.0, q), m, q == 0 ? 1 : 0};
    if (scr.sorted && q == 0)
        cic_binned<kCicPeriodic>(pos, np, L, acc, scr, st);
    else if (scr.sorted)
        cic_binned<kCicPatch>(pos, np, L, acc, scr, st);
    else if (np > 0) // one kernel for every level: few particles are bound by its first fetch
        k_cic_deposit<<<(unsigned)((np + kBlock - 1) / kBlock), kBlock, 0, st>>>(pos, np, L, acc);
    // delta = count / mean - 1, mean = np / (n 2^q)^3 particles per cell
    const double cells_equiv = std::ldexp((double)n * n * n, 3 * q);
    const double scale = np > 0 ? cells_equiv / ((double)np * kCicOne) : 0.0;
    k_cic_finish<<<blocks_for(cells), kBlock, 0, st>>>(acc, cells, scale, delta);
}

// Interleaving pays from about a particle per eight cells on (256^3 cells: 0.19 ms
// for the pass, 0.12 ns less per particle).  For few particles its launch counts:
// 300000 of them on 64^3 cells take 49 us instead of 42 in no order and 35 instead of
// 30 in cell order; 600000 64 instead of 61 and 42 instead of 40, on 32^3 45 instead of
// 53 and 39 instead of 41, on 128^3 101 instead of 128 and 57 instead of 49.
bool cic_gather_lines(long long np, int n) {
    return np >= (1 << 19) && np >= (long long)((size_t)n * n * n / 8);
}

void launch_cic_gather(const double *pos, long long np, const CicLevels &lv, double *lines,
                       unsigned *lines_off, double *out, hipStream_t st) {
    if (np <= 0) return;
    const unsigned nb = (unsigned)((np + kBlock - 1) / kBlock);
    const bool in_place = out < pos + 3 * np && pos < out + 3 * np;
    const size_t cells = (size_t)lv.n * lv.n * lv.n;
    const bool ask = lines && np <= (long long)cells && !in_place; // the device chooses
    if (in_place && np <= (long long)cells) lines = nullptr;
    if (lines) {
        const unsigned ib = std::min((unsigned)kReduceBlocks / 2, blocks_for(cells / 2));
        if (ask)
            k_cic_interleave<true><<<ib, kBlock, 0, st>>>(lv.force[0], cells, lines, pos, np, lv.n,
                                                         lines_off);
        else
            k_cic_interleave<false><<<ib, kBlock, 0, st>>>(lv.force[0], cells, lines, nullptr, 0,
                                                          lv.n, nullptr);
    }
    // where one of two kernels returns at once, at most 65536 blocks do so (196608 idle
    // ones take 80 us)
    const unsigned cap = ask ? 65536 : ~0u;
    if (ask || !(lines || in_place))
        k_cic_gather_parts<<<std::min(3 * nb, cap), kBlock, 0, st>>>(pos, np, nb, lv,
                                                                    ask ? lines_off : nullptr, out);
    if (ask || lines || in_place)
        k_cic_gather_cells<<<std::min(nb, cap), kBlock, 0, st>>>(pos, np, nb, lv, lines,
                                                                ask ? lines_off : nullptr, out);
}

} // namespace ndgp
