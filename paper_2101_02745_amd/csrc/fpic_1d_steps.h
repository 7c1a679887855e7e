// Whole 1D steps in one launch, for boxes (and batches) of at most one
// workgroup per CU (part of fpic_1d.hip).
//
// With one launch per stage and one per reduction, a step of a small box is
// eight launches of 5 to 27 us each that move almost no data: every launch
// starts cold (descriptor, tables, tile, state, one dependent memory round
// trip after another) and a gap follows it.  Here one launch runs
// all steps of a call: a workgroup keeps its tile and directions, one a wave,
// and the stages are separated by a barrier over the grid.  The work split,
// the arithmetic and the order of every sum are those of the stage kernels
// (fpic_1d_body.h) with one direction a wave and every slope stored; results
// are the same bit for bit.
//
// One barrier per stage: instead of a reduction pass, every workgroup sums
// the direction groups' partials of the cells it interpolates from (67 or 69
// columns) straight into its LDS tile.  Partials go to two buffers in turn,
// so a workgroup that runs ahead by one stage overwrites nothing that is
// still read.
//
// What workgroups exchange (partials, particles that leave a tile) goes through
// device-coherent 8-byte accesses (xld, xst), which pass by the XCDs' L2
// caches; no cache is written back or invalidated.  The barrier waits for
// each wave's stores, then counts workgroups in (two levels: 16 workgroups on
// each counter, since the counter's atomics are served one after another).
//
// Step times (us, one launch per stage -> whole steps): see the rule in
// fpic_runtime.cpp.
#pragma once

#include "fpic_1d_body.h"

namespace fpic {

namespace {

typedef const __attribute__((address_space(4))) SimDesc cSimDesc;

typedef __attribute__((address_space(1))) unsigned guint;

// Waits until counter c has reached target; false if the wait was given up.
__device__ __forceinline__ bool reached(const GridBar &b, guint *c, unsigned target)
{
    const unsigned t0 = (unsigned)wall_clock64();
    while ((int)(__hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - target) < 0) {
        if (__builtin_expect((unsigned)wall_clock64() - t0 > b.bar_ticks, 0))
            return false;
        __builtin_amdgcn_s_sleep(1);
    }
    return true;
}

// Barrier number gen (from 1) over the grid; false if the wait was given up.
__device__ __forceinline__ bool grid_sync(const GridBar &b, unsigned gen, int *sflag)
{
    // this wave's stores are in memory before its workgroup counts in
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned nwg = gridDim.x, grp = blockIdx.x / kBarGroup;
        const unsigned ngrp = (nwg + kBarGroup - 1) / kBarGroup;
        const unsigned size = min((unsigned)kBarGroup, nwg - grp * kBarGroup);
        guint *top = (guint *)b.cnt, *mine = (guint *)(b.cnt + kBarStride * (1 + grp));
        if (__hip_atomic_fetch_add(mine, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == gen * size)
            __hip_atomic_fetch_add(top, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *sflag = reached(b, top, gen * ngrp);
    }
    __syncthreads();
    return *sflag != 0;
}

// The workgroups that do a launch's work: this one's number among them (size
// or more: it has nothing to do).
struct Team {
    unsigned rank, size;
};

// The same over a team that is not the whole grid: barrier number gen (from 1)
// of the launch.
__device__ __forceinline__ bool team_sync(const GridBar &b, const Team &t, unsigned gen, int *sflag)
{
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        guint *c = (guint *)(b.cnt + kBarTeam);
        __hip_atomic_fetch_add(c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *sflag = reached(b, c, gen * t.size);
    }
    __syncthreads();
    return *sflag != 0;
}

// Cell of column col of the grid tile from tile0 - sh, periodic.
__device__ __forceinline__ int tile_cell(int cell, int nc)
{
    cell %= nc;
    return cell < 0 ? cell + nc : cell;
}

// LDS of a workgroup, in doubles: grid tile, its edge sums, every wave's
// share (9 components of 64 cells), every wave's edge buffer, the waves'
// direction components, the particle a wave passes on.
constexpr int kPart = 54;      // reals of a particle on its way: state, slope, sum of slopes
// Edge entries of a tile's columns, at most: every (source tile, slot) reaches
// one cell, and the columns repeat a box of one tile of nc cells ceil(columns /
// nc) times (with more tiles they hold fewer: at most 12).
constexpr int kMaxEdge = 24;
constexpr int edge_entries(int sh) { return n_edges(sh) * ((gt_cells(sh) + kMinStepCells - 1) / kMinStepCells); }
static_assert(edge_entries(1) <= kMaxEdge && edge_entries(2) <= kMaxEdge, "no entry is left out");
struct Lds {
    double *Gt, *Ge, *xc, *eb, *v, *pass;
};
__host__ __device__ constexpr int lds_doubles(int nwaves, int sh)
{
    return NG * gt_stride(sh) + NG * kMaxEdge + nwaves * (9 * TILE + 9 * n_edges(sh) + 4 + kPart);
}

// What reaches the columns of the workgroup's tile: the cell of every column,
// and the edge partials (column, source tile, slot) in the order in which
// they are added.
struct Columns {
    int cell[gt_cells(2)];
    int n;                    // edge entries
    int col[kMaxEdge], src[kMaxEdge], slot[kMaxEdge];
};

// The workgroup's grid tile (as in the stage kernels) from the partials of
// the stage before: a thread sums V values, each over the direction groups,
// the loads of G groups of all of them in flight together.  The edge entries
// are values like the others (in the slots that the tile leaves over) and are
// added to their columns in a second pass.
template <int SH>
__device__ __forceinline__ void tile_from_partials(const cSimDesc &S, const double *part, const double *edge,
                                                   const Lds &L, const Columns &C, int nthr)
{
    constexpr int GTC = gt_cells(SH), GTS = gt_stride(SH), NE = n_edges(SH), V = SH == 2 ? 6 : 5, G = 4;
    const int ng = S.ngroup, ntile = S.ntile, ntc = ntile * TILE, ne = C.n;
    const int gpart = NG * ntc, gedge = NG * NE * ntile;
    const int items = NG * (GTC + ne);
#pragma unroll 1
    for (int base = threadIdx.x; base < items; base += V * nthr) {
        int at[V], stride[V];
        const double *pp[V];
        double s[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int idx = min(base + v * nthr, items - 1);  // past the end: the last value again
            if (idx < NG * GTC) {
                const int comp = idx / GTC, col = idx - comp * GTC;
                at[v] = comp * GTS + col;
                pp[v] = part + comp * ntc + C.cell[col];
                stride[v] = gpart;
            } else {
                const int q = idx - NG * GTC, i = q / NG, comp = q - i * NG;
                at[v] = NG * GTS + q;  // Ge follows Gt
                pp[v] = edge + (comp * NE + C.slot[i]) * ntile + C.src[i];
                stride[v] = gedge;
            }
            s[v] = 0.0;
        }
        int g = 0;
#pragma unroll 1
        for (; g + G <= ng; g += G) {
            double x[G][V];
#pragma unroll
            for (int q = 0; q < G; ++q)
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    x[q][v] = xld<true>(pp[v]);
                    pp[v] += stride[v];
                }
#pragma unroll
            for (int q = 0; q < G; ++q)
#pragma unroll
                for (int v = 0; v < V; ++v)
                    s[v] += x[q][v];
        }
#pragma unroll 1
        for (; g < ng; ++g) {
            double x[V];
#pragma unroll
            for (int v = 0; v < V; ++v) {
                x[v] = xld<true>(pp[v]);
                pp[v] += stride[v];
            }
#pragma unroll
            for (int v = 0; v < V; ++v)
                s[v] += x[v];
        }
#pragma unroll
        for (int v = 0; v < V; ++v)
            L.Gt[at[v]] = s[v];
    }
    __syncthreads();
    // one component a thread, so that a column with several entries takes
    // them in order
    if (threadIdx.x < NG)
        for (int i = 0; i < ne; ++i)
            L.Gt[threadIdx.x * GTS + C.col[i]] += L.Ge[i * NG + threadIdx.x];
    __syncthreads();
}

// Shift and fraction of a stage's anchor time (stage mode of step n): where
// its deposit takes the particles.
__device__ __forceinline__ Shift anchor_shift(double vz, int64_t n, int mode, double dt, double dz)
{
    const double t = mode == M_S4 ? stage_time(n + 1, dt, 0.0) : stage_time(n, dt, mode == M_S3 ? 1.0 : 0.5);
    return shift_of(vz, t, dz);
}

// N values of every lane's particle moved by e = 1 or -1 lanes.  The lane at
// the receiving end takes the particle in in (LDS), or, in a box of one tile
// (ring), that of this wave's other end.
template <int N>
__device__ __forceinline__ void move_lanes(double *v, int e, int lane, int nact, bool ring, const double *in)
{
    const int end = e > 0 ? 0 : nact - 1, from = e > 0 ? nact - 1 : 0;
#pragma unroll
    for (int k = 0; k < N; k++) {
        const double x = e > 0 ? lane_below(v[k]) : lane_above(v[k]);
        double w = in[k];
        if (ring)
            w = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v[k]), from),
                                 __builtin_amdgcn_readlane(__double2loint(v[k]), from));
        v[k] = lane == end ? w : x;
    }
}

// A work item: a tile and one direction a wave.
struct Item {
    const cSimDesc *ds;
    int nc, ndir, ntile, tile, group;
    int m, nact, d, nw;   // the lane's cell, active lanes, the wave's direction, waves with one
    bool has, active, first;
    double vx, vy, vz, wN, wNb;
};

template <int SH>
__device__ __forceinline__ void set_item(Item &I, const WorkItem &wi, const SimDesc *sims, const Lds &L,
                                         Columns &C, int wave, int lane, int nwaves)
{
    constexpr int GTC = gt_cells(SH);
    I.ds = (const cSimDesc *)(sims + wi.sim);
    I.nc = I.ds->ncell;
    I.ndir = I.ds->ndir;
    I.ntile = I.ds->ntile;
    I.tile = wi.tile;
    I.group = wi.group;
    const int tile0 = wi.tile * TILE, d0 = wi.group * nwaves;
    I.m = tile0 + lane;
    I.nact = min(TILE, I.nc - tile0);
    I.d = d0 + wave;
    I.nw = min(nwaves, I.ndir - d0);
    I.has = wave < I.nw;
    I.active = I.has && I.m < I.nc;
    I.first = wi.group == 0;  // writes the tile's grid
    I.vx = I.vy = I.vz = I.wN = I.wNb = 0.0;
    if (I.has) {
        I.vx = tld(I.ds->vx, I.d);
        I.vy = tld(I.ds->vy, I.d);
        I.vz = tld(I.ds->vz, I.d);
        I.wN = tld(I.ds->wN, I.d);
        I.wNb = tld(I.ds->wNb, I.d);
    }
    if (lane == 0) {
        L.v[wave * 4 + 0] = 1.0;
        L.v[wave * 4 + 1] = I.vx;
        L.v[wave * 4 + 2] = I.vy;
        L.v[wave * 4 + 3] = I.vz;
    }
    for (int col = threadIdx.x; col < GTC; col += nwaves * TILE)
        C.cell[col] = tile_cell(tile0 - SH + col, I.nc);
    __syncthreads();
    if (threadIdx.x == 0) {
        int n = 0;
        for (int col = 0; col < GTC; ++col) {
            const int t = C.cell[col] / TILE;
            edge_sources(SH, I.nc, I.ntile, t, C.cell[col] - t * TILE, [&](int src, int e) {
                C.col[n] = col;
                C.src[n] = src;
                C.slot[n] = e;
                ++n;
            });
        }
        C.n = n;
    }
    __syncthreads();
}

__device__ __forceinline__ int64_t particle_at(const Item &I, const Shift &s)
{
    int c = I.m - pmod_dbl((double)s.i, I.nc);
    c = c < 0 ? c + I.nc : c;
    return (int64_t)I.d * I.nc + c;
}

// All steps of the launch's work items.  Every wave has one direction of its
// workgroup's tile, a particle a lane.  SHARED false: one item a workgroup, its
// particles in registers: the state, the previous slope and the sum of the
// slopes so far.  When the direction's anchor moves on by a cell from one stage
// to the next, the wave moves its particles by one lane and passes the one at
// the end to the neighbouring tile's wave through memory (xch, two buffers in
// turn); loading and storing them all in every stage, as the stage kernels
// do, took 10.8 us a stage of the 32 x 26 box against 9.3.  SHARED: the team
// takes the items in turn, stage by stage, with their particles in memory
// (slopes in xch; a particle's next stage may be another workgroup's): two
// steps of the 2048 x 64 box, with the host's wait, 700 us by 140 to 190 of its
// 256 workgroups, against 436 by all.  The four stages are one body (mode is
// uniform): a body for each was 36 KB of code a stage, more than the
// instruction cache holds for a step.  Ends early, with sflag 0, where a
// barrier's wait was given up.
template <int SH, bool SHARED>
__device__ __forceinline__ void all_steps(const WorkItem *__restrict__ work, const SimDesc *__restrict__ sims,
                                          int stride, int keep, int nsteps, const GridBar &bar, const Lds &L,
                                          Columns &C, int *sflag, const Team &team, int wave, int lane, int nwaves)
{
    constexpr int GTC = gt_cells(SH), GTS = gt_stride(SH), NE = n_edges(SH);
    Item I;
    double Y[18], kp[18], ks[18];
    Shift sn;
    int move = 0;
    const int lo = SHARED ? (int)team.rank : (int)blockIdx.x, hi = SHARED ? (int)gridDim.x : lo + 1;
    const int inc = SHARED ? (int)team.size : 1;
    int64_t n0 = *((const cSimDesc *)(sims + work[lo].sim))->step;
    if (!SHARED) {
        set_item<SH>(I, work[lo], sims, L, C, wave, lane, nwaves);
        sn = anchor_shift(I.vz, n0, M_S1, I.ds->dt, I.ds->dz);
        const int64_t p = particle_at(I, sn), np = I.ds->np;
        const double *Yp = I.ds->Y;
#pragma unroll
        for (int k = 0; k < 18; k++) {
            Y[k] = I.active ? gld(Yp + k * np + p) : 0.0;
            kp[k] = ks[k] = 0.0;
        }
    }
    // stage it % 4 + 1 of step it / 4; its partials go to buffer it % 2.  The
    // last turn only forms the next step's stage-1 grid.
#pragma unroll 1
    for (int it = 0; it <= 4 * nsteps; ++it) {
        const bool last = it == 4 * nsteps, odd = it & 1;
        const int st = last ? nsteps - 1 : it >> 2, mode = (it & 3) + 1;
        for (int item = lo; item < hi; item += inc) {
            if (SHARED) {
                set_item<SH>(I, work[item], sims, L, C, wave, lane, nwaves);
                n0 = *I.ds->step;
            }
            if (last && !I.first) {
                if (SHARED)
                    continue;
                return;
            }
            const cSimDesc &S = I.ds[(int64_t)st * stride];
            const int64_t n = n0 + (it >> 2), np = S.np;
            const double dt = S.dt, dz = S.dz;
            const int ntc = I.ntile * TILE, tile0 = I.tile * TILE;
            if (SHARED) {
                sn = anchor_shift(I.vz, n, mode, dt, dz);
                const int64_t p = particle_at(I, sn);
                const double *Yp = S.Y, *kx = S.xch;
#pragma unroll
                for (int k = 0; k < 18; k++) {
                    Y[k] = I.active ? xld<true>(Yp + k * np + p) : 0.0;
                    kp[k] = I.active && mode != M_S1 ? xld<true>(kx + k * np + p) : 0.0;
                    ks[k] = I.active && mode != M_S1 ? xld<true>(kx + (18 + k) * np + p) : 0.0;
                }
            }
            const Shift sc = shift_of(I.vz, stage_time(n, dt, mode == M_S1 ? 0.0 : (mode == M_S4 ? 1.0 : 0.5)), dz);
            const int delta = max(-1, min(1, (int)(sn.i - sc.i)));
            // the particle that comes in from the next tile, a real a lane;
            // used after the tile has formed
            const bool moves = !SHARED && move != 0 && I.has && !last;
            double in = 0.0;
            if (moves && I.ntile > 1 && lane < kPart) {
                const int nb = move > 0 ? (I.tile == 0 ? I.ntile - 1 : I.tile - 1)
                                        : (I.tile == I.ntile - 1 ? 0 : I.tile + 1);
                in = xld<true>(S.xch + (((size_t)odd * I.ndir + I.d) * I.ntile + nb) * kPart + lane);
            }
            if (it == 0) {
                const double *gin = S.G[0];
                for (int idx = threadIdx.x; idx < NG * GTC; idx += nwaves * TILE) {
                    const int comp = idx / GTC, col = idx - comp * GTC;
                    L.Gt[comp * GTS + col] = gld(gin + (size_t)comp * I.nc + C.cell[col]);
                }
                __syncthreads();
            } else {
                tile_from_partials<SH>(S, odd ? S.part : S.part2, odd ? S.edge : S.edge2, L, C, nwaves * TILE);
            }
            if (moves) {
                if (lane < kPart)
                    L.pass[lane] = in;
                __builtin_amdgcn_wave_barrier();
                move_lanes<18>(Y, move, lane, I.nact, I.ntile == 1, L.pass);
                if (mode != M_S1) {
                    move_lanes<18>(kp, move, lane, I.nact, I.ntile == 1, L.pass + 18);
                    move_lanes<18>(ks, move, lane, I.nact, I.ntile == 1, L.pass + 36);
                }
            }
            if (last || (keep && I.first && it > 0)) {
                double *G = last ? S.G[4]
                                 : (mode == M_S1 ? S.G[0]
                                                 : (mode == M_S2 ? S.G[1] : (mode == M_S3 ? S.G[2] : S.G[3])));
                for (int k = wave; k < NG; k += nwaves)
                    if (lane < I.nact)
                        gst(G + (size_t)k * I.nc + I.m, L.Gt[k * GTS + lane + SH]);
            }
            if (last) {
                // the boxes' step counters: every workgroup has read them
                if (!SHARED && I.tile == 0 && threadIdx.x == 0)
                    *I.ds->step = n0 + nsteps;
                __syncthreads();
                continue;
            }

            if (I.has) {
                double X[9];
                if (I.active) {
                    double y[18], yn[18];
                    const double a = mode == M_S4 ? dt : 0.5 * dt, h6 = dt / 6.0;
                    if (mode == M_S1) {
#pragma unroll
                        for (int k = 0; k < 18; k++)
                            y[k] = Y[k];
                    } else {
#pragma unroll
                        for (int k = 0; k < 18; k++)
                            y[k] = __builtin_fma(a, kp[k], Y[k]);
                    }
                    double hv[9], hvb[9], Hnn[9];
#pragma unroll
                    for (int k = 0; k < 9; k++) {
                        hv[k] = S.hvac[k];
                        hvb[k] = S.hvacb[k];
                    }
                    gather_hnn<SH>(L.Gt, GTS, lane - delta + SH, sc.phi, I.vx, I.vy, I.vz, Hnn);
                    slope_of(hv, hvb, Hnn, y, kp);
                    if (mode == M_S4) {
#pragma unroll
                        for (int k = 0; k < 18; k++) {
                            const double base = __builtin_fma(h6, ks[k], Y[k]);
                            yn[k] = Y[k] = __builtin_fma(h6, kp[k], base);
                        }
                    } else {
                        const double an = mode == M_S3 ? dt : 0.5 * dt;
#pragma unroll
                        for (int k = 0; k < 18; k++) {
                            yn[k] = __builtin_fma(an, kp[k], Y[k]);
                            ks[k] = mode == M_S1 ? kp[k] : ks[k] + 2.0 * kp[k];
                        }
                    }
                    if (SHARED || keep || it == 4 * nsteps - 1) {
                        const int64_t p = particle_at(I, sn);
                        if (mode == M_S4) {
                            double *out = S.Yout;
#pragma unroll
                            for (int k = 0; k < 18; k++)
                                xst<SHARED>(out + k * np + p, Y[k]);
                        } else if (keep) {
                            store_slope(mode == M_S1 ? S.K1 : (mode == M_S2 ? S.K2 : S.K3), np, p, kp);
                        }
                        if (SHARED) {
                            double *kx = S.xch;
#pragma unroll
                            for (int k = 0; k < 18; k++) {
                                xst<true>(kx + k * np + p, kp[k]);
                                xst<true>(kx + (18 + k) * np + p, ks[k]);
                            }
                        }
                    }
#pragma unroll
                    for (int k = 0; k < 9; k++)
                        X[k] = source_comp(k, I.wN, yn[k], I.wNb, yn[9 + k]);
                } else {
#pragma unroll
                    for (int k = 0; k < 9; k++)
                        X[k] = 0.0;
                }
                double xc[9];
                deposit_share<SH>(X, sn.phi, lane, I.nact, xc, L.eb + wave * 9 * NE);
#pragma unroll
                for (int k = 0; k < 9; k++)
                    L.xc[(wave * 9 + k) * TILE + lane] = xc[k];
            }
            if (!SHARED) {
                // the next stage's anchor; the particle that leaves the tile
                // with it
                const int nmode = (mode & 3) + 1;
                const Shift sx = anchor_shift(I.vz, n0 + ((it + 1) >> 2), nmode, dt, dz);
                move = __builtin_amdgcn_readfirstlane((int)(sx.i - sn.i));
                sn = sx;
                if (move != 0 && I.has && I.ntile > 1) {
                    if (lane == (move > 0 ? I.nact - 1 : 0)) {
#pragma unroll
                        for (int k = 0; k < 18; k++) {
                            L.pass[k] = Y[k];
                            L.pass[18 + k] = kp[k];
                            L.pass[36 + k] = ks[k];
                        }
                    }
                    __builtin_amdgcn_wave_barrier();
                    if (lane < kPart)
                        xst<true>(S.xch + (((size_t)!odd * I.ndir + I.d) * I.ntile + I.tile) * kPart + lane,
                                  L.pass[lane]);
                }
            }
            __syncthreads();
            // the moments of the workgroup's directions, in wave order; a
            // product is rounded before it is added, as where a wave
            // accumulates its own.  Component k of all four groups by wave k;
            // the ninth (and the rest, with fewer waves) a group a wave, the
            // edges by the last wave.
            double *part = (odd ? S.part2 : S.part) + (size_t)I.group * NG * ntc + tile0 + lane;
            {
                double a0 = 0.0, ax = 0.0, ay = 0.0, az = 0.0;
#pragma unroll 4
                for (int w = 0; w < I.nw; ++w) {
                    const double x = L.xc[(w * 9 + wave) * TILE + lane];
                    a0 += x;
                    ax += __builtin_fma(L.v[w * 4 + 1], x, 0.0);
                    ay += __builtin_fma(L.v[w * 4 + 2], x, 0.0);
                    az += __builtin_fma(L.v[w * 4 + 3], x, 0.0);
                }
                double *o = part + (size_t)wave * ntc;
                xst<true>(o, a0);
                xst<true>(o + (size_t)9 * ntc, ax);
                xst<true>(o + (size_t)18 * ntc, ay);
                xst<true>(o + (size_t)27 * ntc, az);
            }
#pragma unroll 1
            for (int q = 4 * nwaves + wave; q < NG; q += nwaves) {
                const int k = q >> 2, g = q & 3;
                double a = 0.0;
#pragma unroll 4
                for (int w = 0; w < I.nw; ++w)
                    a += __builtin_fma(L.v[w * 4 + g], L.xc[(w * 9 + k) * TILE + lane], 0.0);
                xst<true>(part + (size_t)(9 * g + k) * ntc, a);
            }
            if (wave == nwaves - 1) {
                double *edge = odd ? S.edge2 : S.edge;
#pragma unroll 1
                for (int q = lane; q < NE * NG; q += TILE) {
                    const int e = q / NG, r = q - e * NG, comp = r % 9, grp = r / 9;
                    double t = 0.0;
#pragma unroll 4
                    for (int w = 0; w < I.nw; ++w)
                        t += __builtin_fma(L.v[w * 4 + grp], L.eb[(w * NE + e) * 9 + comp], 0.0);
                    xst<true>(edge + (((size_t)I.group * NG + r) * NE + e) * I.ntile + I.tile, t);
                }
            }
            if (SHARED)
                __syncthreads();  // the next item overwrites the LDS
        }
        // (a team waits after the last turn too: its first workgroup then
        // writes the step counters)
        if (SHARED ? !team_sync(bar, team, (unsigned)it + 1u, sflag)
                   : !last && !grid_sync(bar, bar.gen + (unsigned)it + 1u, sflag))
            return;
    }
}

// After a wait that was given up: the failure words, then NaN in every state
// that the launch was to return (by each workgroup that gives up, the last of
// them last), so that what is read from the context before the host has looked
// at its word cannot pass for a result.
__device__ __forceinline__ void give_up(const GridBar &b, const WorkItem *__restrict__ work,
                                        const SimDesc *__restrict__ sims, int end)
{
    if (threadIdx.x == 0) {
        __hip_atomic_store((guint *)(b.cnt + kBarBad), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(b.failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    for (int q = 0; q < (int)gridDim.x; ++q) {
        if (work[q].tile != 0 || work[q].group != 0)
            continue;
        const cSimDesc *S = (const cSimDesc *)(sims + work[q].sim) + end;
        double *Y = S->Yout;
        for (int64_t i = threadIdx.x; i < 18 * S->np; i += blockDim.x)
            xst<true>(Y + i, __longlong_as_double(0x7ff8000000000000ll));
    }
}

// The workgroups that do the launch's work: all of them, once every one is
// resident, or those that are when a wait for that has lasted arrive_ticks.
//
// Every workgroup counts itself in, which numbers it.  The last one decides for
// the whole grid.  One that has waited arrive_ticks decides for those that have
// counted in by then (the first decision holds): the others, when they start,
// end at once, so that no wait depends on a workgroup that cannot start.
// Launches of this process that run at the same time fit the chip together
// (steps_reserve on the host), so that this is for other kernels that hold CUs
// for as long.  The decision is one word: the launch's number, then the team's
// size (kDeciding: being made).  After a wait that an earlier launch has given
// up, nobody does anything.
constexpr unsigned kSizeBits = 10, kDeciding = (1u << kSizeBits) - 1;
static_assert(kMaxStepWgs < kDeciding, "a team's size fits its bits");

__device__ __forceinline__ Team team_of(const GridBar &b, int *sflag)
{
    if (threadIdx.x == 0) {
        guint *arrive = (guint *)(b.cnt + kBarArrive), *mode = (guint *)(b.cnt + kBarMode);
        const unsigned tag = (b.launch + 1u) << kSizeBits, base = b.launch * gridDim.x;
        // size of the team, 0: undecided (mode's value in cur)
        unsigned cur;
        auto decided = [&]() {
            cur = __hip_atomic_load(mode, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return (cur ^ tag) >> kSizeBits ? 0u : cur & kDeciding;
        };
        auto decide = [&](unsigned size) {
            return __hip_atomic_compare_exchange_strong(mode, &cur, tag | size, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT);
        };
        const unsigned bad = __hip_atomic_load((guint *)(b.cnt + kBarBad), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned rank = __hip_atomic_fetch_add(arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - base;
        if (rank + 1u == gridDim.x && decided() == 0)
            decide(gridDim.x);
        const unsigned long long t0 = wall_clock64();
        unsigned size;
        while ((size = decided()) == 0 || size == kDeciding) {
            if (size == 0 && wall_clock64() - t0 >= b.arrive_ticks && decide(kDeciding)) {
                size = __hip_atomic_load(arrive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - base;
                // the team's counter is clear before anyone counts on it
                __hip_atomic_store((guint *)(b.cnt + kBarTeam), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __hip_atomic_store(mode, tag | size, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __builtin_amdgcn_s_sleep(1);
        }
        sflag[0] = (int)rank;
        sflag[1] = bad ? 0 : (int)size;
    }
    __syncthreads();
    const Team t = {(unsigned)__builtin_amdgcn_readfirstlane(sflag[0]),
                    (unsigned)__builtin_amdgcn_readfirstlane(sflag[1])};
    __syncthreads();
    return t;
}

template <int SH>
__global__ void __launch_bounds__(MAX_WAVES * TILE)
steps1d_kernel(const WorkItem *__restrict__ work, const SimDesc *__restrict__ sims, int stride, int keep,
               int nsteps, GridBar bar)
{
    extern __shared__ double smem[];
    __shared__ int sflag, tflag[2];
    __shared__ Columns C;
    const int lane = threadIdx.x & (TILE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / TILE);
    const int nwaves = blockDim.x / TILE;
    Lds L;
    L.Gt = smem;
    L.Ge = L.Gt + NG * gt_stride(SH);
    L.xc = L.Ge + NG * kMaxEdge;
    L.eb = L.xc + nwaves * 9 * TILE;
    L.v = L.eb + nwaves * 9 * n_edges(SH);
    L.pass = L.v + nwaves * 4 + wave * kPart;  // this wave's
    const Team team = team_of(bar, tflag);
    if (team.rank >= team.size)
        return;
    if (team.size == gridDim.x) {
        all_steps<SH, false>(work, sims, stride, keep, nsteps, bar, L, C, &sflag, team, wave, lane, nwaves);
    } else {
        all_steps<SH, true>(work, sims, stride, keep, nsteps, bar, L, C, &sflag, team, wave, lane, nwaves);
        if (sflag != 0 && team.rank == 0) {
            // the step counters, and the barriers that the next launch counts on
            for (int q = threadIdx.x; q < (int)gridDim.x; q += blockDim.x)
                if (work[q].tile == 0 && work[q].group == 0)
                    *sims[work[q].sim].step += nsteps;
            const unsigned nwg = gridDim.x, ngrp = (nwg + kBarGroup - 1) / kBarGroup, nbar = 4u * nsteps;
            for (unsigned g = threadIdx.x; g < ngrp; g += blockDim.x)
                __hip_atomic_fetch_add((guint *)(bar.cnt + kBarStride * (1 + g)),
                                       nbar * min((unsigned)kBarGroup, nwg - g * kBarGroup), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            if (threadIdx.x == 0)
                __hip_atomic_fetch_add((guint *)bar.cnt, nbar * ngrp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (sflag == 0)  // (as the latest barrier left it; every launch has one)
        give_up(bar, work, sims, (nsteps - 1) * stride);
}

size_t steps1d_smem(int waves, int shape) { return lds_doubles(waves, shape) * sizeof(double); }

}  // namespace

bool steps1d_fits(int nwork, int waves, int shape)
{
    int dev = 0, cus = 0, per = 0;
    const size_t smem = steps1d_smem(waves, shape);
    const void *f = shape == 2 ? (const void *)steps1d_kernel<2> : (const void *)steps1d_kernel<1>;
    const bool ok = nwork <= kMaxStepWgs && smem <= 160 * 1024 && hipGetDevice(&dev) == hipSuccess &&
                    hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
                    hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, f, waves * TILE, smem) == hipSuccess;
    (void)hipGetLastError();
    return ok && (int64_t)per * cus >= nwork;
}

hipError_t launch_steps1d(const WorkItem *work, int nwork, const SimDesc *sims, int stride, int keep,
                          int waves, int shape, int nsteps, const GridBar &bar, hipStream_t s)
{
    if (nsteps < 1 || nwork < 1 || nwork > kMaxStepWgs)
        return hipErrorInvalidValue;
    const dim3 grid(nwork), block(waves * TILE);
    const size_t smem = steps1d_smem(waves, shape);
    if (shape == 2)
        steps1d_kernel<2><<<grid, block, smem, s>>>(work, sims, stride, keep, nsteps, bar);
    else
        steps1d_kernel<1><<<grid, block, smem, s>>>(work, sims, stride, keep, nsteps, bar);
    return hipGetLastError();
}

}  // namespace fpic
