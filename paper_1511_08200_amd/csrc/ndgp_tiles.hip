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
// V(2,2) cycle, us per level (per-colour launches -> this): 64^3 50 -> 35, 32^3
// 50 -> 22, 16^3 33 -> 20, and 9 for the coarsest level's own launch.  Four launches
// per level is near the floor that launches set; at 64^3 the restricting sweep (14.6
// us; 8 at 32^3, 6 at 16^3) is bound by the arithmetic of its halo, 4.4 times the
// tile's own.
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

// The same for the levels of a refinement (padded, FP64): the finest with its fixed
// ghost shell, the coarse ones with ghosts that follow the interior (dyn), held
// cells kept.  A cell that changes rewrites its ghosts (write_owned_ghosts) in the
// step that stores it, from the level's hat values held in LDS beside the field.
// V(2,2) cycle of a 128^3 refinement's coarse levels, us (per-colour launches -> this):
// 64^3 60 -> 53, 32^3 55 -> 33, and 62 (one workgroup from 16^3 down) -> 30 + 16 for
// the coarsest level's own launch.
template <int TILE, int NS, bool PRO, bool REST, int NT>
__global__ void __launch_bounds__(NT)
k_tile_dir(TileDirArgs a) {
    constexpr int H = 2 * NS + (REST ? 2 : 0);
    constexpr int W = TILE + 2 * H, HX = W / 2, PL = W * HX;
    constexpr int NC = TILE / 2 + 2, NE = W / 2 + 2;
    __shared__ double U[2][W * PL];
    __shared__ double HL[2][W * PL]; // hat of this level (dyn)
    __shared__ double E[PRO ? NE * NE * NE : 1];
    __shared__ double HC[REST ? NC * NC * NC : 1];
    __shared__ double RS[REST ? TILE * TILE * TILE : 1];

    const int lg = a.lg, n = 1 << lg, pitch = n + 2;
    const int nt = n / TILE;
    const int tile = xcd_local_id(blockIdx.x, gridDim.x);
    const int x0 = (tile % nt) * TILE - H, y0 = (tile / nt % nt) * TILE - H,
              z0 = (tile / (nt * nt)) * TILE - H;
    const int tid = threadIdx.x;
    // a tile whose region reaches the shell (else no ghost is met)
    const bool edge = x0 < 0 || y0 < 0 || z0 < 0 || x0 + W > n || y0 + W > n || z0 + W > n;
    const bool dyn = a.dyn && edge;
    auto inside = [&](int x, int y, int z) { // local coordinates
        return (unsigned)(x0 + x) < (unsigned)n && (unsigned)(y0 + y) < (unsigned)n &&
               (unsigned)(z0 + z) < (unsigned)n;
    };
    auto in_shell = [&](int x, int y, int z) {
        return (unsigned)(x0 + x + 1) < (unsigned)pitch && (unsigned)(y0 + y + 1) < (unsigned)pitch &&
               (unsigned)(z0 + z + 1) < (unsigned)pitch;
    };
    auto padded = [&](int x, int y, int z) {
        return ((z0 + z + 1) * pitch + y0 + y + 1) * pitch + x0 + x + 1;
    };
    auto natural = [&](int x, int y, int z) { return (((z0 + z) << lg) + y0 + y) * n + x0 + x; };
    auto slot = [&](int x, int y, int z) { return z * PL + y * HX + (x >> 1); };
    // f(x, y, z, factor) of every ghost of interior cell (x, y, z) inside the region
    auto for_ghosts = [&](int x, int y, int z, auto f) {
        const int gx = x0 + x, gy = y0 + y, gz = z0 + z;
        const int sx = gx == 0 ? -1 : gx == n - 1 ? 1 : 0, sy = gy == 0 ? -1 : gy == n - 1 ? 1 : 0,
                  sz = gz == 0 ? -1 : gz == n - 1 ? 1 : 0;
        if (!(sx | sy | sz)) return;
#pragma unroll
        for (int m = 1; m < 8; ++m) {
            if (((m & 1) && !sx) || ((m & 2) && !sy) || ((m & 4) && !sz)) continue;
            const int qx = x + (m & 1 ? sx : 0), qy = y + (m & 2 ? sy : 0), qz = z + (m & 4 ? sz : 0);
            if ((unsigned)qx >= (unsigned)W || (unsigned)qy >= (unsigned)W || (unsigned)qz >= (unsigned)W)
                continue;
            const int d = (m & 1) + ((m >> 1) & 1) + ((m >> 2) & 1);
            f(qx, qy, qz, d == 1 ? -1.0 / 3.0 : (d == 2 ? 1.0 / 9.0 : -1.0 / 27.0));
        }
    };
    auto set_ghosts = [&](int x, int y, int z, double val) {
        const double e = val - HL[(x + y + z) & 1][slot(x, y, z)];
        for_ghosts(x, y, z, [&](int qx, int qy, int qz, double f) {
            const int c = (qx + qy + qz) & 1, q = slot(qx, qy, qz);
            U[c][q] = HL[c][q] + f * e;
        });
    };

    const int lgc = lg - 1, nc = n >> 1, pc = nc + 2;
    auto coarse_padded = [&](int I, int J, int K) { return ((K + 1) * pc + J + 1) * pc + I + 1; };
    if constexpr (PRO) // the coarse correction under the region (where cells use it)
        for (int q = tid; q < NE * NE * NE; q += NT) {
            const int I = x0 / 2 - 1 + q % NE, J = y0 / 2 - 1 + q / NE % NE,
                      K = z0 / 2 - 1 + q / (NE * NE);
            const bool on = (unsigned)(I + 1) < (unsigned)pc && (unsigned)(J + 1) < (unsigned)pc &&
                            (unsigned)(K + 1) < (unsigned)pc;
            const int g = on ? coarse_padded(I, J, K) : 0;
            E[q] = on ? a.phi_c[g] - a.hat_c[g] : 0.0;
        }
    if (dyn)
        for (int q = tid; q < W * W * W; q += NT) {
            const int x = q % W, y = q / W % W, z = q / (W * W);
            if (in_shell(x, y, z)) HL[(x + y + z) & 1][slot(x, y, z)] = a.hat[padded(x, y, z)];
        }
    if (PRO || dyn) __syncthreads();
    for (int q = tid; q < W * W * W; q += NT) {
        const int x = q % W, y = q / W % W, z = q / (W * W);
        if (!in_shell(x, y, z)) continue;
        const bool in = inside(x, y, z);
        if (PRO && dyn && !in) continue; // written by its cell, whose value changes
        double v = a.pin[padded(x, y, z)];
        if constexpr (PRO) {
            if (in && (!a.mask || a.mask[natural(x, y, z)])) {
                const int sx = (x & 1) ? 1 : -1, sy = (y & 1) ? 1 : -1, sz = (z & 1) ? 1 : -1;
                const int e0 = ((z / 2 + 1) * NE + y / 2 + 1) * NE + x / 2 + 1;
                double acc = 0.0;
#pragma unroll
                for (int cz = 0; cz < 2; ++cz)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            const double wt = (i ? 0.25 : 0.75) * (b ? 0.25 : 0.75) * (cz ? 0.25 : 0.75);
                            acc = fma(wt, E[e0 + (cz * sz * NE + b * sy) * NE + i * sx], acc);
                        }
                v = v + acc;
            }
            if (dyn) set_ghosts(x, y, z, v);
        }
        U[(x + y + z) & 1][slot(x, y, z)] = v;
    }
    __syncthreads();

    auto stencil = [&](const double *own, const double *other, int x, int y, int z, double v[19]) {
        const int xp = (x + 1) >> 1, xm = xp - 1, s = x >> 1;
        const double *A = own + z * PL + y * HX, *O = other + z * PL + y * HX;
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
        double nv[each], src[each];
        bool on[each];
#pragma unroll
        for (int e = 0; e < each; ++e) { // the sources first: one wait for memory
            const int t = tid + e * NT, y = lo + t / (S / 2) % S, z = lo + t / (S / 2 * S);
            const int x = lo + 2 * (t % (S / 2)) + ((lo + y + z + c) & 1);
            on[e] = t < items && inside(x, y, z);
            if (on[e]) {
                src[e] = a.s[natural(x, y, z)];
                if (a.mask) on[e] = a.mask[natural(x, y, z)] != 0; // a held cell is kept
            }
        }
#pragma unroll
        for (int e = 0; e < each; ++e) {
            const int t = tid + e * NT, y = lo + t / (S / 2) % S, z = lo + t / (S / 2 * S);
            const int x = lo + 2 * (t % (S / 2)) + ((lo + y + z + c) & 1);
            if (on[e]) {
                double v[19];
                stencil(U[c], U[1 - c], x, y, z, v);
                unsigned ev = 0;
                nv[e] = relax_cell(v, src[e], a.al, a.w, ev);
                // a halo cell's events are counted by the workgroup that owns it
                if (ev && (unsigned)(x - H) < (unsigned)TILE && (unsigned)(y - H) < (unsigned)TILE &&
                    (unsigned)(z - H) < (unsigned)TILE)
                    events += ev;
            }
            __builtin_amdgcn_sched_barrier(0); // one cell at a time: no spills
        }
        __syncthreads(); // every read sees the values of the half sweep's start
#pragma unroll
        for (int e = 0; e < each; ++e) {
            const int t = tid + e * NT, y = lo + t / (S / 2) % S, z = lo + t / (S / 2 * S);
            const int x = lo + 2 * (t % (S / 2)) + ((lo + y + z + c) & 1);
            if (on[e]) {
                U[c][slot(x, y, z)] = nv[e];
                if (dyn) set_ghosts(x, y, z, nv[e]);
            }
        }
        __syncthreads();
    };
    half_sweep(Int<0>{});
    half_sweep(Int<1>{});
    if constexpr (NS == 2) {
        half_sweep(Int<2>{});
        half_sweep(Int<3>{});
    }

    // the tile itself, and the ghosts of its cells
    for (int q = tid; q < TILE * TILE * TILE; q += NT) {
        const int x = H + q % TILE, y = H + q / TILE % TILE, z = H + q / (TILE * TILE);
        a.pout[padded(x, y, z)] = U[(x + y + z) & 1][slot(x, y, z)];
        if (dyn)
            for_ghosts(x, y, z, [&](int qx, int qy, int qz, double) {
                a.pout[padded(qx, qy, qz)] = U[(qx + qy + qz) & 1][slot(qx, qy, qz)];
            });
    }

    if constexpr (REST) {
        // mean of the children, and the coarse level's own ghosts where they are met
        const int I0 = (x0 + H) / 2 - 1, J0 = (y0 + H) / 2 - 1, K0 = (z0 + H) / 2 - 1;
        for (int q = tid; q < NC * NC * NC; q += NT) {
            const int I = I0 + q % NC, J = J0 + q / NC % NC, K = K0 + q / (NC * NC);
            if ((unsigned)I < (unsigned)nc && (unsigned)J < (unsigned)nc && (unsigned)K < (unsigned)nc) {
                const int x = 2 * I - x0, y = 2 * J - y0, z = 2 * K - z0;
                double sum = 0.0;
#pragma unroll
                for (int ch = 0; ch < 8; ++ch) {
                    const int cx = x + (ch & 1), cy = y + (ch >> 1 & 1), cz = z + (ch >> 2);
                    sum += U[(cx + cy + cz) & 1][slot(cx, cy, cz)];
                }
                HC[q] = sum * 0.125;
            } else {
                HC[q] = a.hat_out[coarse_padded(I, J, K)];
            }
        }
        // the residual of each of the tile's cells, children of a coarse cell together
        for (int q = tid; q < TILE * TILE * TILE; q += NT) {
            const int ch = q & 7, cell = q >> 3;
            const int x = H + 2 * (cell % (TILE / 2)) + (ch & 1),
                      y = H + 2 * (cell / (TILE / 2) % (TILE / 2)) + (ch >> 1 & 1),
                      z = H + 2 * (cell / (TILE / 2 * TILE / 2)) + (ch >> 2);
            const int c = (x + y + z) & 1, g = natural(x, y, z);
            double v[19];
            stencil(U[c], U[1 - c], x, y, z, v);
            RS[q] = a.mask && !a.mask[g] ? 0.0 : a.s[g] - apply_L(stencil_terms(v), a.al);
        }
        __syncthreads();
        for (int q = tid; q < TILE * TILE * TILE / 8; q += NT) {
            const int I = q % (TILE / 2), J = q / (TILE / 2) % (TILE / 2), K = q / (TILE / 2 * TILE / 2);
            double sr = 0.0;
#pragma unroll
            for (int ch = 0; ch < 8; ++ch) sr += RS[q * 8 + ch];
            const double sc = sr * 0.5; // 4 * mean: the coarse cell is twice as wide
            const int o = ((K + 1) * NC + J + 1) * NC + I + 1;
            constexpr int dy = NC, dz = NC * NC;
            const double v[19] = {
                HC[o], HC[o + 1], HC[o - 1], HC[o + dy], HC[o - dy], HC[o + dz], HC[o - dz],
                HC[o + 1 + dy], HC[o + 1 - dy], HC[o - 1 + dy], HC[o - 1 - dy],
                HC[o + 1 + dz], HC[o + 1 - dz], HC[o - 1 + dz], HC[o - 1 - dz],
                HC[o + dy + dz], HC[o + dy - dz], HC[o - dy + dz], HC[o - dy - dz]};
            const int gi = I0 + 1 + I, gj = J0 + 1 + J, gk = K0 + 1 + K;
            a.s_out[((gk << lgc) + gj) * nc + gi] = apply_L(stencil_terms(v), a.al_c) + sc;
            a.hat_out[coarse_padded(gi, gj, gk)] = v[0];
            a.phi_out[coarse_padded(gi, gj, gk)] = v[0];
            // no correction yet: the coarse field's ghosts are its hat's
            const int sx = gi == 0 ? -1 : gi == nc - 1 ? 1 : 0, sy = gj == 0 ? -1 : gj == nc - 1 ? 1 : 0,
                      sz = gk == 0 ? -1 : gk == nc - 1 ? 1 : 0;
            if (sx | sy | sz)
                for (int m = 1; m < 8; ++m) {
                    if (((m & 1) && !sx) || ((m & 2) && !sy) || ((m & 4) && !sz)) continue;
                    const int ex = m & 1 ? sx : 0, ey = m & 2 ? sy : 0, ez = m & 4 ? sz : 0;
                    a.phi_out[coarse_padded(gi + ex, gj + ey, gk + ez)] =
                        HC[o + (ez * NC + ey) * NC + ex];
                }
        }
    }
    if (events) flush_events(a.events, events);
}

template <int TILE, int NT>
void tile_dir_launch(const TileDirArgs &a, int sweeps, bool pro, bool rest, hipStream_t st) {
    const int nt = (1 << a.lg) / TILE;
    const unsigned blocks = (unsigned)(nt * nt * nt);
    if (sweeps == 2) {
        if (rest) k_tile_dir<TILE, 2, false, true, NT><<<blocks, NT, 0, st>>>(a);
        else if (pro) k_tile_dir<TILE, 2, true, false, NT><<<blocks, NT, 0, st>>>(a);
        else k_tile_dir<TILE, 2, false, false, NT><<<blocks, NT, 0, st>>>(a);
    } else {
        if (rest) k_tile_dir<TILE, 1, false, true, NT><<<blocks, NT, 0, st>>>(a);
        else if (pro) k_tile_dir<TILE, 1, true, false, NT><<<blocks, NT, 0, st>>>(a);
        else k_tile_dir<TILE, 1, false, false, NT><<<blocks, NT, 0, st>>>(a);
    }
}

} // namespace

void launch_tile(const TileArgs<double> &a, int sweeps, bool pro, bool rest, hipStream_t st) {
    tile_level<TileField>(a, sweeps, pro, rest, st);
}

void launch_tile(const TileArgs<float> &a, int sweeps, bool pro, bool rest, hipStream_t st) {
    tile_level<TileCorrection>(a, sweeps, pro, rest, st);
}

void launch_tile_dir(const TileDirArgs &a, int sweeps, bool pro, bool rest, hipStream_t st) {
    if (a.lg <= 5) tile_dir_launch<4, 256>(a, sweeps, pro, rest, st);
    else tile_dir_launch<8, 512>(a, sweeps, pro, rest, st);
}

} // namespace ndgp
