// ndgp_tiles.hip -- the small levels of a periodic V-cycle (16^3 to 64^3 cells),
// tile by tile in LDS.
//
// On these levels every launch is bound by its latency: a per-colour half sweep
// takes 4.7 us whatever it does, and a level needed eleven dependent launches
// per cycle (50 us); the levels from 16^3 down, solved by one workgroup in LDS,
// took 43 us, nearly all of it 16^3's arithmetic on one compute unit.  Here a
// launch does a whole red-black sweep, and the first one going up also adds the
// coarse-grid correction (on load), the last one going down also restricts the
// swept field and its residual and forms the FAS coarse source.  A workgroup
// loads a 4^3 or 8^3 tile with a halo as wide as the launch reaches (two cells per
// sweep, two more for the restriction) and relaxes it over a region that
// shrinks by one cell per half sweep.  Halo cells are relaxed by several
// workgroups; each gets the same arithmetic on the same values, in the order of
// the per-level kernels (k_smooth_half, k_restrict_residual, k_coarse_source,
// k_prolong8 and their FP32 counterparts), so the result is bit for bit theirs.
//
// V(2,2) cycle, us per level (before -> now): 64^3 50 -> 35, 32^3 50 -> 20, 16^3
// 33 -> 19, and 9 for the coarsest level's own launch.  Four launches per level
// is near the floor that launches set; at 64^3 the restricting sweep (14.6 us)
// is bound by the arithmetic of its halo, 4.4 times the tile's own.
//
// LDS keeps both colours apart, so that lanes on consecutive cells of one
// colour touch consecutive words.

#include "ndgp_tiles.h"

namespace ndgp {
namespace {

using namespace dev;

template <class P, int kTile, int NS, bool PRO, bool REST, int NT>
__global__ void __launch_bounds__(NT)
k_tile(TileArgs<typename P::T> a) {
    using T = typename P::T;
    constexpr int H = 2 * NS + (REST ? 2 : 0); // halo of the tile
    constexpr int W = kTile + 2 * H, HX = W / 2, PL = W * HX;
    constexpr int NC = kTile / 2 + 2;          // coarse cells per side, one-cell halo
    constexpr int NE = W / 2 + 2;              // coarse cells under the region, one-cell halo
    __shared__ T U[2][W * PL];
    __shared__ T B[P::two ? 2 : 1][P::two ? W * PL : 1]; // the static field of the correction
    __shared__ T E[PRO ? NE * NE * NE : 1];
    __shared__ T HC[REST ? NC * NC * NC : 1], BC[REST && P::two ? NC * NC * NC : 1];
    __shared__ T RS[REST ? kTile * kTile * kTile : 1];

    const int lg = a.lg, n = 1 << lg, m = n - 1;
    const int nt = n / kTile;
    const int tile = xcd_local_id(blockIdx.x, gridDim.x);
    // the region's lower corner (even in every axis: local parity is the colour)
    const int x0 = (tile % nt) * kTile - H, y0 = (tile / nt % nt) * kTile - H,
              z0 = (tile / (nt * nt)) * kTile - H;
    const int tid = threadIdx.x;
    auto at = [&](int x, int y, int z) {
        return (((((z0 + z) & m) << lg) | ((y0 + y) & m)) << lg) | ((x0 + x) & m);
    };

    if constexpr (PRO) { // the coarse correction under the region
        const int lgc = lg - 1, mc = (n >> 1) - 1;
        for (int q = tid; q < NE * NE * NE; q += NT) {
            const int I = x0 / 2 - 1 + q % NE, J = y0 / 2 - 1 + q / NE % NE,
                      K = z0 / 2 - 1 + q / (NE * NE);
            const int g = ((((K & mc) << lgc) | (J & mc)) << lgc) | (I & mc);
            E[q] = a.phi_c[g] - a.hat_c[g];
        }
        __syncthreads();
    }
    // pairs of cells (columns 2j, 2j + 1 of a row: one of each colour)
    using Pair = typename P::Pair;
    for (int q = tid; q < W * PL; q += NT) {
        const int j = q % HX, y = q / HX % W, z = q / PL;
        const int g = at(2 * j, y, z);
        const int c = (y + z) & 1; // colour of column 2j
        T v[2] = {T(0), T(0)};
        if (!a.from_zero) {
            const Pair p = *reinterpret_cast<const Pair *>(a.pin + g);
            v[0] = p.x;
            v[1] = p.y;
        }
        if constexpr (PRO) {
            const int sy = (y & 1) ? 1 : -1, sz = (z & 1) ? 1 : -1;
            const int e0 = ((z / 2 + 1) * NE + y / 2 + 1) * NE + j + 1;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int sx = i ? 1 : -1;
                T acc = T(0);
#pragma unroll
                for (int cz = 0; cz < 2; ++cz)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int x = 0; x < 2; ++x) {
                            const T wt = T((x ? 0.25 : 0.75) * (b ? 0.25 : 0.75) * (cz ? 0.25 : 0.75));
                            acc = P::fma_(wt, E[e0 + (cz * sz * NE + b * sy) * NE + x * sx], acc);
                        }
                v[i] += acc;
            }
        }
        U[c][q] = v[0];
        U[1 - c][q] = v[1];
        if constexpr (P::two) {
            const Pair p = *reinterpret_cast<const Pair *>(a.base + g);
            B[c][q] = p.x;
            B[1 - c][q] = p.y;
        }
    }
    if constexpr (REST && P::two) {
        const int lgc = lg - 1, mc = (n >> 1) - 1;
        for (int q = tid; q < NC * NC * NC; q += NT) {
            const int I = (x0 + H) / 2 - 1 + q % NC, J = (y0 + H) / 2 - 1 + q / NC % NC,
                      K = (z0 + H) / 2 - 1 + q / (NC * NC);
            BC[q] = a.base_c[((((K & mc) << lgc) | (J & mc)) << lgc) | (I & mc)];
        }
    }
    __syncthreads();

    // the 19-point stencil of cell (x, y, z) of colour c
    auto stencil = [&](const T *own, const T *other, int x, int y, int z, T v[19]) {
        const int xp = (x + 1) >> 1, xm = xp - 1, s = x >> 1;
        const T *A = own + z * PL + y * HX, *O = other + z * PL + y * HX;
        v[0] = A[s];
        v[1] = O[xp];
        v[2] = O[xm];
        v[3] = O[HX + s];
        v[4] = O[s - HX];
        v[5] = O[PL + s];
        v[6] = O[s - PL];
        v[7] = A[HX + xp];
        v[8] = A[xp - HX];
        v[9] = A[HX + xm];
        v[10] = A[xm - HX];
        v[11] = A[PL + xp];
        v[12] = A[xp - PL];
        v[13] = A[PL + xm];
        v[14] = A[xm - PL];
        v[15] = A[PL + HX + s];
        v[16] = A[HX - PL + s];
        v[17] = A[PL - HX + s];
        v[18] = A[s - PL - HX];
    };

    unsigned events = 0;
    auto half_sweep = [&](auto hc) {
        constexpr int h = decltype(hc)::value, c = h & 1;
        constexpr int lo = h + 1, S = W - 2 * lo, items = S * S * S / 2;
        constexpr int each = (items + NT - 1) / NT;
        T nv[each], src[each];
#pragma unroll
        for (int e = 0; e < each; ++e) { // the sources first: one wait for memory
            const int t = tid + e * NT, y = lo + t / (S / 2) % S, z = lo + t / (S / 2 * S);
            const int x = lo + 2 * (t % (S / 2)) + ((lo + y + z + c) & 1);
            if (t < items) src[e] = a.s[at(x, y, z)];
        }
#pragma unroll
        for (int e = 0; e < each; ++e) {
            const int t = tid + e * NT, y = lo + t / (S / 2) % S, z = lo + t / (S / 2 * S);
            const int x = lo + 2 * (t % (S / 2)) + ((lo + y + z + c) & 1);
            if (t < items) {
                T v[19], vb[19];
                stencil(U[c], U[1 - c], x, y, z, v);
                if constexpr (P::two) stencil(B[c], B[1 - c], x, y, z, vb);
                unsigned ev = 0;
                nv[e] = P::relax(v, vb, src[e], a.al, a.w, ev);
                // a halo cell's events are counted by the workgroup that owns it
                if (ev && (unsigned)(x - H) < (unsigned)kTile &&
                    (unsigned)(y - H) < (unsigned)kTile && (unsigned)(z - H) < (unsigned)kTile)
                    events += ev;
            }
            __builtin_amdgcn_sched_barrier(0); // one cell at a time: no spills
        }
        __syncthreads(); // every read sees the values of the half sweep's start
#pragma unroll
        for (int e = 0; e < each; ++e) {
            const int t = tid + e * NT, y = lo + t / (S / 2) % S, z = lo + t / (S / 2 * S);
            const int x = lo + 2 * (t % (S / 2)) + ((lo + y + z + c) & 1);
            if (t < items) U[c][z * PL + y * HX + (x >> 1)] = nv[e];
        }
        __syncthreads();
    };
    half_sweep(Int<0>{});
    half_sweep(Int<1>{});
    if constexpr (NS == 2) {
        half_sweep(Int<2>{});
        half_sweep(Int<3>{});
    }

    // the tile itself
    constexpr int pairs = kTile * kTile * kTile / 2;
    for (int q = tid; q < pairs; q += NT) {
        const int j = q % (kTile / 2), y = q / (kTile / 2) % kTile, z = q / (kTile / 2 * kTile);
        const int l = (z + H) * PL + (y + H) * HX + j + H / 2, c = (y + z) & 1;
        Pair p;
        p.x = U[c][l];
        p.y = U[1 - c][l];
        *reinterpret_cast<Pair *>(a.pout + at(2 * j + H, y + H, z + H)) = p;
    }

    if constexpr (REST) {
        // mean of the children: the tile's coarse cells and one around them
        auto value = [&](int x, int y, int z) {
            return U[(x + y + z) & 1][z * PL + y * HX + (x >> 1)];
        };
        for (int q = tid; q < NC * NC * NC; q += NT) {
            const int x = H - 2 + 2 * (q % NC), y = H - 2 + 2 * (q / NC % NC),
                      z = H - 2 + 2 * (q / (NC * NC));
            T sum = T(0);
#pragma unroll
            for (int ch = 0; ch < 8; ++ch) sum += value(x + (ch & 1), y + (ch >> 1 & 1), z + (ch >> 2));
            HC[q] = sum * T(0.125);
        }
        // the residual of each of the tile's cells, children of a coarse cell together
        for (int q = tid; q < kTile * kTile * kTile; q += NT) {
            const int ch = q & 7, cell = q >> 3;
            const int x = H + 2 * (cell % (kTile / 2)) + (ch & 1),
                      y = H + 2 * (cell / (kTile / 2) % (kTile / 2)) + (ch >> 1 & 1),
                      z = H + 2 * (cell / (kTile / 2 * kTile / 2)) + (ch >> 2);
            const int c = (x + y + z) & 1;
            T v[19], vb[19];
            stencil(U[c], U[1 - c], x, y, z, v);
            if constexpr (P::two) stencil(B[c], B[1 - c], x, y, z, vb);
            RS[q] = a.s[at(x, y, z)] - P::apply(v, vb, a.al);
        }
        __syncthreads();
        for (int q = tid; q < pairs / 4; q += NT) { // (kTile / 2)^3 coarse cells
            const int I = q % (kTile / 2), J = q / (kTile / 2) % (kTile / 2),
                      K = q / (kTile / 2 * kTile / 2);
            T sr = T(0);
#pragma unroll
            for (int ch = 0; ch < 8; ++ch) sr += RS[q * 8 + ch];
            const T sc = sr * T(0.5); // 4 * mean: the coarse cell is twice as wide
            auto coarse = [&](const T *f, T v[19]) {
                const T *o = f + ((K + 1) * NC + J + 1) * NC + I + 1;
                constexpr int dy = NC, dz = NC * NC;
                const int off[19] = {0, 1, -1, dy, -dy, dz, -dz,
                                     1 + dy, 1 - dy, -1 + dy, -1 - dy,
                                     1 + dz, 1 - dz, -1 + dz, -1 - dz,
                                     dy + dz, dy - dz, -dy + dz, -dy - dz};
#pragma unroll
                for (int k = 0; k < 19; ++k) v[k] = o[off[k]];
            };
            T v[19], vb[19];
            coarse(HC, v);
            if constexpr (P::two) coarse(BC, vb);
            const int lgc = lg - 1;
            const int g = ((((z0 + H) / 2 + K) << lgc | ((y0 + H) / 2 + J)) << lgc) |
                          ((x0 + H) / 2 + I);
            a.s_out[g] = P::apply(v, vb, a.al_c) + sc;
            a.hat_out[g] = v[0];
            a.phi_out[g] = v[0];
        }
    }
    if (events) flush_events(a.events, events);
}

template <class P, int TILE, int NT>
void tile_launch(const TileArgs<typename P::T> &a, int sweeps, bool pro, bool rest,
                 hipStream_t st) {
    const int nt = (1 << a.lg) / TILE;
    const unsigned blocks = (unsigned)(nt * nt * nt);
    if (sweeps == 2) {
        if (rest) k_tile<P, TILE, 2, false, true, NT><<<blocks, NT, 0, st>>>(a);
        else if (pro) k_tile<P, TILE, 2, true, false, NT><<<blocks, NT, 0, st>>>(a);
        else k_tile<P, TILE, 2, false, false, NT><<<blocks, NT, 0, st>>>(a);
    } else {
        if (rest) k_tile<P, TILE, 1, false, true, NT><<<blocks, NT, 0, st>>>(a);
        else if (pro) k_tile<P, TILE, 1, true, false, NT><<<blocks, NT, 0, st>>>(a);
        else k_tile<P, TILE, 1, false, false, NT><<<blocks, NT, 0, st>>>(a);
    }
}

// 4^3 tiles on the smallest levels, so that their few cells spread over the chip
// (32^3: 512 workgroups; restricting sweep 7.4 us, 9.1 with 64 workgroups of 8^3),
// 8^3 on 64^3 (512 workgroups too; smaller tiles relax more halo)
template <class P>
void tile_level(const TileArgs<typename P::T> &a, int sweeps, bool pro, bool rest,
                hipStream_t st) {
    if (a.lg <= 5) tile_launch<P, 4, 256>(a, sweeps, pro, rest, st);
    else tile_launch<P, 8, 512>(a, sweeps, pro, rest, st);
}

} // namespace

void launch_tile(const TileArgs<double> &a, int sweeps, bool pro, bool rest, hipStream_t st) {
    tile_level<TileField>(a, sweeps, pro, rest, st);
}

void launch_tile(const TileArgs<float> &a, int sweeps, bool pro, bool rest, hipStream_t st) {
    tile_level<TileCorrection>(a, sweeps, pro, rest, st);
}

} // namespace ndgp
