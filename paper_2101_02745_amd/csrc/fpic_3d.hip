// 3D periodic boxes: two kernels per Runge-Kutta stage.
//
// particle kernel (a workgroup = one x-row of current cells and a group of
// directions, lane = x): forms the stage state, interpolates the combined
// moments at the particle's current position with the trilinear
// cloud-in-cell weights (y and z first, from the four neighbouring grid rows
// staged in LDS, then x from the lane one to the right), builds H and Hbar,
// the commutator slopes and the next stage state, and writes that state's
// deposit source X = (N/dV) rho - (Nbar/dV) rhobar^* (its traceless part: 8
// reals per particle, see NXT below).
//
// deposit kernel (one wave = one x-row of destination cells, all directions, or
// in boxes of few rows a quarter of them, in a fixed order):
// every cell pulls X from the eight particles whose next-stage positions
// straddle it (four rows in y and z, then the lane one to the left in x)
// with the same weights, and accumulates the combined moments (32 traceless
// components; 36 for the moments diagnostic) in registers.  Each cell is
// written once, without atomics: bitwise reproducible.
//
// Positions are implicit as in 1D: particle (d, c) is at cell c shifted by
// floor(Omega_a t / dx_a) along each axis with fraction Omega_a t / dx_a minus
// that, t = n dt + c_s dt.  Along an axis with one cell the particle stays in
// cell 0 with weight 1.  A row of at most 64 cells is one wave (lane = x);
// a longer row is cut into segments with halo lanes (XRow below).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "fpic_3d.h"
#include "fpic_device.h"
#include "fpic_internal.h"

namespace fpic3d {

using fpic::commutator;
using fpic::fail;
using fpic::gld;
using fpic::gst;
using fpic::source_comp;
using fpic::stage_time;
using fpic::tld;
using fpic::wsum2;
using fpic::wsum3;

constexpr int NG = 36;
constexpr int W = 64;

// Parameters of one direction for a fused linear stage, computed once per
// stage by dirtab3f_kernel: its integer shift at the next stage time, the
// offset of its current lower cell from the next one in x, its current
// cloud-in-cell fractions (x, and the y/z weights of the four gather rows),
// and the deposit coefficients of the next stage: c[4 q + g] = w_q m_g, with
// w_q the y/z weight of destination row q and m = (1, v_x, v_y, v_z).
struct FDir {
    int32_t rxn, ryn, rzn, dxs;
    int32_t cls, pad_[3];
    double fx;
    double wyz[4];
    double fxn;     // fxn and c are contiguous: the deposit reads them as 17 reals
    double c[16];
    double vx, vy, vz, wN, wNb, pad2_[2];
};
constexpr int FDIR_DEP = 9;  // offset of fxn in an FDir, in doubles

struct Desc3 {
    int32_t n[3];    // nx, ny, nz
    int32_t ndir;
    int64_t ncell, np;
    double dt, dx[3];
    double hvac[9];         // constant part of H (vacuum + matter), packed
    double hvacb[9];        // of Hbar before conjugation (vacuum - matter)
    const double *v[3];     // [ndir] direction components
    const double *wN, *wNb; // [ndir] N/dV, Nbar/dV
    const double *Nw, *Nbw; // [ndir] N, Nbar
    double *Y, *K1, *K2, *K3;
    double *X;              // [9][ndir][ncell] deposit sources (stages: 8 traceless)
    double *G[2];           // [36][ncell] (stages: 32 traceless): stage s reads G[(s-1)&1]
    int64_t *step;
    int32_t shape;          // shape-function order: 1 linear, 2 quadratic
    int32_t pad_;
    // fused linear stages: [4][NGT][ncell] deposit partials, slot q = 2 cz + cy
    // holding a workgroup's contributions to the row (cy, cz) above its own;
    // rowmap[b] is the x-row (y + ny z) of workgroup b
    double *P4;
    const int32_t *rowmap;
    // fused linear stages: per-direction parameters of the current stage
    // (FDir, written by dirtab3f_kernel), the class order of the directions
    // and the end of each class in it
    FDir *ftab;
    int32_t *forder;
    int32_t *fcls_end;  // [9]
};

// integer shift (mod n) and fraction along one axis; one-cell axes: (0, 0)
__device__ __forceinline__ void axis_shift(double v, double t, double dx, int n, int *r, double *phi)
{
#pragma clang fp contract(off)
    if (n == 1) {
        *r = 0;
        *phi = 0.0;
        return;
    }
    const double u = (v * t) / dx;
    const double fl = floor(u);
    *phi = u - fl;
    const double nd = (double)n;
    double q = fl - nd * floor(fl / nd);
    if (q < 0.0)
        q += nd;
    if (q >= nd)
        q -= nd;
    *r = (int)q;
}

// Slopes in memory: fpic::NK reals per particle (components 0 and 9 are
// the negated sums of the next two and are not stored).
__device__ __forceinline__ int kslot(int c) { return c < 9 ? c - 1 : c - 2; }

// The particle streams of the fused kernels (state, slopes) are read and
// written with the streaming (nontemporal) policy: a wave touches a whole
// x-row, and the arrays (gigabytes) are far larger than the Infinity Cache, so
// caching them only evicts the grid rows that are re-read (the 64^3 x 92 box:
// 10.24 -> 9.60 ms per step; rows of 50 and 40 cells, too, are 1 % faster).
// The separate kernels stream only rows that are whole cache lines (streams()
// below).  The 1D kernels keep most streams cacheable: there neighbouring
// tiles share cache lines of the rotated rows, and full streaming was much
// slower.
//
// NT: streaming (nontemporal) loads and stores
template <bool NT>
__device__ __forceinline__ double pld(const double *p)
{
    return NT ? fpic::gld_nt(p) : gld(p);
}
template <bool NT>
__device__ __forceinline__ void pst(double *p, double v)
{
    if (NT)
        fpic::gst_nt(p, v);
    else
        gst(p, v);
}

template <bool NT>
__device__ __forceinline__ void load_slope(const double *K, int64_t np, int64_t p, bool active, double k[18])
{
#pragma unroll
    for (int c = 1; c < 18; c++)
        if (c != 9)
            k[c] = active ? pld<NT>(K + kslot(c) * np + p) : 0.0;
    k[0] = -(k[1] + k[2]);
    k[9] = -(k[10] + k[11]);
}

__device__ __forceinline__ double lane_get(double v, int src)
{
    return __shfl(v, src, W);
}

// x-rows and waves.  In a box with nx <= 64 a wave holds a whole x-row:
// lane x is cell x and the neighbours of lane x are the lanes x +- 1 mod nx.
// A longer row is cut into segments of sw = 64 - HL - HR cells; lane j of
// segment s holds cell (s sw - HL + j) mod nx, the lanes [HL, HL + width)
// own the segment's cells, and the HL lanes below and HR lanes above them
// only supply neighbour values: the cell to the right for the linear
// interpolation in x (HR = 1), the particle to the left for the linear
// deposit (HL = 1), both for the quadratic shape.  Every lane of a segment
// holds a real cell, so its loads need no mask.
__host__ __device__ constexpr int xsegs(int nx, int sw) { return nx <= W ? 1 : (nx + sw - 1) / sw; }

struct XRow {
    int x;            // the lane's cell (0 in lanes past a whole row)
    bool own;         // the lane updates / writes its cell
    bool valid;       // the lane holds a cell of the row (its values are used)
    int left, right;  // lanes holding cells x - 1 and x + 1
};

template <int HL, int HR>
__device__ __forceinline__ XRow xrow(int nx, int seg, int lane)
{
    XRow r;
    if (nx <= W) {
        r.valid = r.own = lane < nx;
        r.x = r.own ? lane : 0;
        r.left = (lane + nx - 1) % nx;
        r.right = (lane + 1) % nx;
    } else {
        constexpr int sw = W - HL - HR;
        const int x0 = seg * sw;
        int x = x0 - HL + lane;  // in [-1, 2 nx)
        x = (x < 0) ? x + nx : ((x >= nx) ? x - nx : x);
        r.x = x;
        r.valid = true;
        r.own = lane >= HL && lane < HL + min(sw, nx - x0);
        r.left = lane - 1;   // owners never take lane -1 or 64
        r.right = lane + 1;
    }
    return r;
}

// Stage deposits carry the traceless part of each 3x3 source matrix: the
// interpolated Hamiltonian is needed only up to a multiple of the identity,
// which commutes with every state and leaves both commutators unchanged.
// Per particle the source X = (N/dV) rho - (Nbar/dV) rhobar^* is stored as
// NXT = 8 reals (x11 - x00, x22 - x00 and the six off-diagonal reals), and
// the stage grids hold NGT = 32 components (A, B_x, B_y, B_z, eight each);
// the moments diagnostic deposits all nine components of its sources.
constexpr int NXT = 8, NGT = 4 * NXT;

template <bool NT>
__device__ __forceinline__ void store_source(const Desc3 &S, int64_t p, double wN, double wNb,
                                             const double yn[18])
{
    double x[9];
#pragma unroll
    for (int k = 0; k < 9; k++)
        x[k] = source_comp(k, wN, yn[k], wNb, yn[9 + k]);
    pst<NT>(S.X + p, x[1] - x[0]);
    pst<NT>(S.X + S.np + p, x[2] - x[0]);
#pragma unroll
    for (int k = 3; k < 9; k++)
        pst<NT>(S.X + (k - 1) * S.np + p, x[k]);
}

// MODE 1..4: Runge-Kutta stages; 5: deposit sources of the current state.
//
// A workgroup owns one row (y, z) of *current* lower cells and a group of
// directions (waves x dpw); for direction d, lane x takes the particle whose
// lower cell at the stage time is (x, y, z), i.e. the one stored at cell
// (x, y, z) minus the direction's integer shift.  Every particle of the
// workgroup then interpolates from the same four grid rows (y or y + 1,
// z or z + 1), which are staged in LDS once per workgroup; the particle data
// of each direction is one contiguous row, rotated in x.  MODE 5 has no
// interpolation and takes the particles in storage order.
constexpr int MAX_WAVES3 = 8;

// The work item of block b of n: consecutive blocks go to the eight XCDs in
// turn, so every XCD takes a run of consecutive items.  For the segments of
// long rows, whose ends share cache lines (150 x 40 x 32 cells x 24 directions:
// 3.74 -> 3.44 ms per step), and for deposits of one row a workgroup, which
// share source rows (60 x 50 x 50 x 40 quadratic 4.74 -> 4.41 ms).  Whole rows
// of the particle kernels share few lines, patches of 2 x 2 whole rows in the
// deposits less than single ones, and neighbours on all XCDs at once use the
// memory channels better (50 x 44 x 36 x 24 quadratic 2.02 ms, particle kernels
// in runs 2.07; 64^3 x 92 quadratic 14.75 ms, deposits in runs 14.93).
constexpr int XCDS = 8;
__device__ __forceinline__ int xcd_item(int b, int n)
{
    const int x = b % XCDS, i = b / XCDS, q = n / XCDS, r = n % XCDS;
    return x * q + min(x, r) + i;
}

template <int MODE, bool NT>
__global__ void __launch_bounds__(MAX_WAVES3 * W)
particle3d_kernel(const Desc3 *__restrict__ dp, int dpw, int nitems)
{
    __shared__ double Gt[MODE == 5 ? 1 : 4 * NGT * W];  // [row q = 2 cz + cy][comp][x]
    const Desc3 S = *dp;
    const int lane = threadIdx.x & (W - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / W);
    const int nwaves = blockDim.x / W;
    const int item = S.n[0] > W ? xcd_item(blockIdx.x, nitems) : (int)blockIdx.x;
    if (item >= nitems)
        return;  // whole workgroup: uniform
    const int nx = S.n[0], ny = S.n[1], nz = S.n[2];
    const int nseg = xsegs(nx, W - 1);
    const int nrs = ny * nz * nseg;
    const int rs = item % nrs, grp = item / nrs;
    const int row = rs / nseg, seg = rs % nseg;
    const int y0 = row % ny, z0 = row / ny;
    const XRow xr = xrow<0, 1>(nx, seg, lane);
    const bool active = xr.own;
    const int64_t n = *S.step;
    const double dt = S.dt;
    double t_cur = 0.0;
    if (MODE == 2 || MODE == 3)
        t_cur = stage_time(n, dt, 0.5);
    else if (MODE == 4)
        t_cur = stage_time(n, dt, 1.0);
    else
        t_cur = stage_time(n, dt, 0.0);
    const double *Gin = S.G[(MODE - 1) & 1];
    const double *Kp = (MODE == 2) ? S.K1 : (MODE == 3) ? S.K2 : S.K3;
    const int dbeg = (grp * nwaves + wave) * dpw, dend = min(dbeg + dpw, S.ndir);
    const int right = xr.right;

    if (MODE != 5) {
        // column j: the cell of lane j
        const int ncol = min(nx, W), xbase = (nx <= W) ? 0 : seg * (W - 1);
        for (int idx = threadIdx.x; idx < 4 * NGT * ncol; idx += blockDim.x) {
            const int j = idx % ncol, t = idx / ncol;
            const int comp = t % NGT, q = t / NGT;
            int yy = y0 + (q & 1), zz = z0 + (q >> 1);
            yy = (yy >= ny) ? yy - ny : yy;
            zz = (zz >= nz) ? zz - nz : zz;
            int x = xbase + j;
            x = (x >= nx) ? x - nx : x;
            Gt[(q * NGT + comp) * W + j] = gld(Gin + (int64_t)comp * S.ncell + ((int64_t)zz * ny + yy) * nx + x);
        }
        __syncthreads();
    }

    for (int d = dbeg; d < dend; ++d) {
        const double vx = tld(S.v[0], d), vy = tld(S.v[1], d), vz = tld(S.v[2], d);
        const double wN = tld(S.wN, d), wNb = tld(S.wNb, d);
        int rx = 0, ry = 0, rz = 0;
        double fx = 0.0, fy = 0.0, fz = 0.0;
        int64_t c;
        if (MODE == 5) {
            c = (int64_t)row * nx + xr.x;
        } else {
            axis_shift(vx, t_cur, S.dx[0], nx, &rx, &fx);
            axis_shift(vy, t_cur, S.dx[1], ny, &ry, &fy);
            axis_shift(vz, t_cur, S.dx[2], nz, &rz, &fz);
            int cx = xr.x - rx, cy = y0 - ry, cz = z0 - rz;
            cx = (cx < 0) ? cx + nx : cx;
            cy = (cy < 0) ? cy + ny : cy;
            cz = (cz < 0) ? cz + nz : cz;
            c = ((int64_t)cz * ny + cy) * nx + (active ? cx : 0);
        }
        const int64_t p = (int64_t)d * S.ncell + c;
        double Y[18];
#pragma unroll
        for (int k = 0; k < 18; k++)
            Y[k] = active ? pld<NT>(S.Y + k * S.np + p) : 0.0;
        double yn[18];
        if (MODE == 5) {
#pragma unroll
            for (int k = 0; k < 18; k++)
                yn[k] = Y[k];
        } else {
            // Hnn = A - (vx B_x + vy B_y + vz B_z), its ee entry 0: y/z
            // interpolation from the four staged rows, one group of 8
            // traceless components (A, B_x, B_y, B_z) at a time with its
            // factor, then x with the lane to the right (periodic in x) once
            // for the sum of the groups
            double wyz[4];
#pragma unroll
            for (int cz = 0; cz < 2; cz++)
#pragma unroll
                for (int cy = 0; cy < 2; cy++)
                    wyz[2 * cz + cy] = (cy ? fy : 1.0 - fy) * (cz ? fz : 1.0 - fz);
            double r[NXT];
#pragma unroll
            for (int k = 0; k < NXT; k++)
                r[k] = 0.0;
#pragma unroll 1
            for (int grp4 = 0; grp4 < 4; grp4++) {
                const double coef = (grp4 == 0) ? 1.0 : (grp4 == 1) ? -vx : (grp4 == 2) ? -vy : -vz;
                const double *g = Gt + NXT * grp4 * W + lane;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const double c = coef * wyz[q];
#pragma unroll
                    for (int k = 0; k < NXT; k++)
                        r[k] += c * (xr.valid ? g[(q * NGT + k) * W] : 0.0);
                }
            }
            double Hnn[9];
            Hnn[0] = 0.0;
#pragma unroll
            for (int k = 0; k < NXT; k++)
                Hnn[k + 1] = (1.0 - fx) * r[k] + fx * lane_get(r[k], right);
            const double a = (MODE == 4) ? dt : 0.5 * dt;
            double yv[18], base[18];
            if (MODE == 1) {
#pragma unroll
                for (int k = 0; k < 18; k++)
                    yv[k] = base[k] = Y[k];
            } else if (MODE == 4) {
                const double h6 = dt / 6.0;
                double k1[18], k2[18], k3[18];
                load_slope<NT>(S.K1, S.np, p, active, k1);
                load_slope<NT>(S.K2, S.np, p, active, k2);
                load_slope<NT>(S.K3, S.np, p, active, k3);
#pragma unroll
                for (int k = 0; k < 18; k++) {
                    yv[k] = Y[k] + dt * k3[k];
                    const double ks = (k1[k] + 2.0 * k2[k]) + 2.0 * k3[k];
                    base[k] = Y[k] + h6 * ks;
                }
            } else {
                double kp[18];
                load_slope<NT>(Kp, S.np, p, active, kp);
#pragma unroll
                for (int k = 0; k < 18; k++) {
                    yv[k] = Y[k] + a * kp[k];
                    base[k] = Y[k];
                }
            }
            double H[9], Hb[9], kk[18];
#pragma unroll
            for (int k = 0; k < 9; k++) {
                H[k] = S.hvac[k] + Hnn[k];
                const double hb = S.hvacb[k] - Hnn[k];
                Hb[k] = (k == 4 || k == 6 || k == 8) ? -hb : hb;
            }
            commutator(H, yv, kk);
            commutator(Hb, yv + 9, kk + 9);
            if (MODE == 4) {
                const double h6 = dt / 6.0;
#pragma unroll
                for (int k = 0; k < 18; k++) {
                    yn[k] = base[k] + h6 * kk[k];
                    if (active)
                        pst<NT>(S.Y + k * S.np + p, yn[k]);
                }
            } else {
                double *Ko = (MODE == 1) ? S.K1 : (MODE == 2) ? S.K2 : S.K3;
                const double an = (MODE == 3) ? dt : 0.5 * dt;
#pragma unroll
                for (int k = 0; k < 18; k++) {
                    if (active && k != 0 && k != 9)
                        pst<NT>(Ko + kslot(k) * S.np + p, kk[k]);
                    yn[k] = base[k] + an * kk[k];
                }
            }
        }
        if (active)
            store_source<NT>(S, p, wN, wNb, yn);
    }
}

// Deposit of the sources at the positions of time t = (n + cnext) dt
// (cnext_num / 2 steps after step n's start; 2 means the next step).
// Each wave owns one x-row of destination cells and sweeps its directions
// in ascending order; per direction it interpolates the sources of the four
// rows in y and z, then in x with the lane to the left (accumulate).  The
// loop is software-pipelined: the 4 NC source values of direction d + 1
// (four rows, NC components) are loaded while direction d is summed.  NC is
// NXT (traceless stage sources, grid of NGT components) or 9 (moments, grid
// of 36).
template <int NC>
struct Pull {
    double X[NC];      // sources interpolated in y and z at the lane's x
    double fx, vx, vy, vz;
};

// One direction's components and interpolation fractions, and its 4 NC raw
// source values for the wave's row at the lane's cell xc (lanes past a whole
// row load a cell of the row that is never used).
template <int NC>
struct DepDir {
    double vx, vy, vz, fx, fy, fz;
    double raw[4 * NC];  // [2 cz + cy][NC]
};

template <int NC>
__device__ __forceinline__ void dep_load(const Desc3 &S, int d, double t, int y, int z, int xc,
                                         DepDir<NC> &o)
{
    const int nx = S.n[0], ny = S.n[1], nz = S.n[2];
    o.vx = tld(S.v[0], d);
    o.vy = tld(S.v[1], d);
    o.vz = tld(S.v[2], d);
    int rx, ry, rz;
    axis_shift(o.vx, t, S.dx[0], nx, &rx, &o.fx);
    axis_shift(o.vy, t, S.dx[1], ny, &ry, &o.fy);
    axis_shift(o.vz, t, S.dx[2], nz, &rz, &o.fz);
    // the same for the whole wave: row addresses in scalar registers
    rx = __builtin_amdgcn_readfirstlane(rx);
    ry = __builtin_amdgcn_readfirstlane(ry);
    rz = __builtin_amdgcn_readfirstlane(rz);
    int xs = xc - rx;
    xs = (xs < 0) ? xs + nx : xs;
#pragma unroll
    for (int cz = 0; cz < 2; cz++)
#pragma unroll
        for (int cy = 0; cy < 2; cy++) {
            int yy = y - ry - cy, zz = z - rz - cz;
            yy = (yy < 0) ? yy + ny : yy;
            yy = (yy < 0) ? yy + ny : yy;
            zz = (zz < 0) ? zz + nz : zz;
            zz = (zz < 0) ? zz + nz : zz;
            const double *xp = S.X + (int64_t)d * S.ncell + ((int64_t)zz * ny + yy) * nx;
#pragma unroll
            for (int k = 0; k < NC; k++)
                o.raw[(cz * 2 + cy) * NC + k] = gld(xp + (int64_t)k * S.np + xs);
        }
}

// y/z interpolation of one direction's raw sources (rows in the order
// cz, cy; inactive lanes take 0)
template <int NC>
__device__ __forceinline__ void pull_dir(const DepDir<NC> &c, bool active, Pull<NC> &o)
{
    o.vx = c.vx;
    o.vy = c.vy;
    o.vz = c.vz;
    o.fx = c.fx;
#pragma unroll
    for (int k = 0; k < NC; k++)
        o.X[k] = 0.0;
#pragma unroll
    for (int cz = 0; cz < 2; cz++)
#pragma unroll
        for (int cy = 0; cy < 2; cy++) {
            const double w = (cy ? c.fy : 1.0 - c.fy) * (cz ? c.fz : 1.0 - c.fz);
#pragma unroll
            for (int k = 0; k < NC; k++)
                o.X[k] += w * (active ? c.raw[(cz * 2 + cy) * NC + k] : 0.0);
        }
}

template <int NC>
__device__ __forceinline__ void accumulate(const Pull<NC> &o, int left, double acc[4 * NC])
{
#pragma unroll
    for (int k = 0; k < NC; k++) {
        const double xl = lane_get(o.X[k], left);
        const double xc = wsum2(1.0 - o.fx, o.X[k], o.fx, xl);
        acc[k] += xc;
        acc[NC + k] += o.vx * xc;
        acc[2 * NC + k] += o.vy * xc;
        acc[3 * NC + k] += o.vz * xc;
    }
}

// A deposit workgroup has four waves.  In a box with many rows it covers a
// patch of 2 x 2 destination rows, one wave per row; its waves sweep the
// directions in the same order, so the source rows they share (a patch of
// 3 x 3 rows per direction) are mostly read from memory once.  With fewer rows
// the waves would be too few to keep enough loads in flight: then the four waves
// share a row (DS = 4), each sweeping a run of the directions, and their sums
// are added in the order of the runs.
constexpr int DEP_WAVES = 4;
template <int DS>
constexpr int dep_py() { return DS == 1 ? 2 : 1; }
template <int DS>
constexpr int dep_pz() { return DS == 1 ? 2 : 1; }

// the wave's row, x-segment and run of directions [d0, d1); none: d0 = d1
struct DepWave {
    int row, y, z, seg, slice, d0, d1;
    bool any;  // the row exists
};
template <int DS>
__device__ __forceinline__ DepWave dep_wave(int ny, int nz, int nseg, int ndir)
{
    constexpr int PY = dep_py<DS>(), PZ = dep_pz<DS>(), ROWS = PY * PZ;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / W);
    const int bi = nseg > 1 || DS > 1 ? xcd_item(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int patch = bi / nseg, npy = (ny + PY - 1) / PY;
    DepWave o;
    o.seg = bi % nseg;
    o.row = wave % ROWS;
    o.slice = wave / ROWS;
    o.y = (patch % npy) * PY + o.row % PY;
    o.z = (patch / npy) * PZ + o.row / PY;
    o.any = o.y < ny && o.z < nz;
    o.d0 = o.any ? (int)((int64_t)ndir * o.slice / DS) : 0;
    o.d1 = o.any ? (int)((int64_t)ndir * (o.slice + 1) / DS) : 0;
    return o;
}

// adds the sums of a row's waves; false in all but the first of them
template <int DS, int NA>
__device__ __forceinline__ bool dep_join(const DepWave &w, int lane, double acc[NA])
{
    if (DS == 1)
        return w.any;
    constexpr int ROWS = dep_py<DS>() * dep_pz<DS>();
    __shared__ double sh[DS == 1 ? 1 : (DS - 1) * ROWS * NA * W];
    if (w.slice > 0)
#pragma unroll
        for (int q = 0; q < NA; q++)
            sh[(((w.slice - 1) * ROWS + w.row) * NA + q) * W + lane] = acc[q];
    __syncthreads();
    if (w.slice > 0)
        return false;
    for (int t = 0; t < DS - 1; t++)
#pragma unroll
        for (int q = 0; q < NA; q++)
            acc[q] += sh[((t * ROWS + w.row) * NA + q) * W + lane];
    return w.any;
}

template <int NC, int DS>
__global__ void __launch_bounds__(DEP_WAVES * W)
deposit3d_kernel(const Desc3 *__restrict__ dp, int half_steps, int out_buf)
{
    const Desc3 S = *dp;
    const int lane = threadIdx.x & (W - 1);
    const int nx = S.n[0], ny = S.n[1], nz = S.n[2];
    const DepWave dw = dep_wave<DS>(ny, nz, xsegs(nx, W - 1), S.ndir);
    const int y = dw.y, z = dw.z, seg = dw.seg;
    const XRow xr = xrow<1, 0>(nx, seg, lane);
    const int64_t n0 = *S.step;
    // half_steps: 0 -> t_n, 1 -> t_n + dt/2, 2 -> t_n + dt (stage 4 of step
    // n), 3 -> first stage of step n + 1
    double t;
    if (half_steps == 3)
        t = stage_time(n0 + 1, S.dt, 0.0);
    else
        t = stage_time(n0, S.dt, 0.5 * half_steps);
    const int left = xr.left;
    double acc[4 * NC];
#pragma unroll
    for (int q = 0; q < 4 * NC; q++)
        acc[q] = 0.0;
    DepDir<NC> nxt;
    if (dw.d0 < dw.d1)
        dep_load<NC>(S, dw.d0, t, y, z, xr.x, nxt);
    for (int d = dw.d0; d < dw.d1; ++d) {
        const DepDir<NC> cur = nxt;
        if (d + 1 < dw.d1)
            dep_load<NC>(S, d + 1, t, y, z, xr.x, nxt);
        Pull<NC> a;
        pull_dir<NC>(cur, xr.valid, a);
        accumulate<NC>(a, left, acc);
    }
    if (!dep_join<DS, 4 * NC>(dw, lane, acc))
        return;
    if (xr.own) {
        double *G = out_buf ? S.G[1] : S.G[0];  // (no dynamic index into the descriptor)
        const int64_t cell = ((int64_t)z * ny + y) * nx + xr.x;
#pragma unroll
        for (int q = 0; q < 4 * NC; q++)
            gst(G + (int64_t)q * S.ncell + cell, acc[q]);
    }
}

// Whether the separate kernels read and write the particles with the streaming
// policy: rows of one wave and whole 128-byte lines (64^3 x 92 linear 12.55 ->
// 12.37 ms per step).  Otherwise neighbouring waves share the lines at the ends
// of their rows or segments, which then stay in L2 until both have used them
// (with segments on the same XCD, see xcd_item): 150 x 40 x 32 cells x 24
// directions 3.74 -> 3.09 ms per step (streaming, 3.43), 130 x 40 x 40 x 92
// 16.4 -> 13.5 ms, 100 x 40 x 40 x 24 quadratic 3.85 -> 3.55 ms, 50 x 44 x 36 x
// 24 quadratic 2.04 -> 2.02 ms.
static bool streams(const Desc3 &h) { return h.n[0] <= W && h.n[0] % 16 == 0; }

// Waves that share a destination row in the deposits (full: of the moments'
// nine components): four up to 1.25 times the rows that the chip holds with one
// wave each, above that one.  With one wave a row the registers allow 12 waves
// of the quadratic stage kernel and 8 of the others on each of 256 CUs (with
// four waves a row, 8 of each).  Per step, one wave a row against four: 12 x 10
// x 14 cells x 50 directions quadratic (140 rows) 1010 -> 456 us, 70 x 8 x 8 x
// 12 (128) 161 -> 106, 50 x 44 x 36 x 24 quadratic (1584) 1908 -> 1849, 32 x 48
// x 48 x 92 (2304) 4459 -> 4205, quadratic 6497 -> 6116, 128 x 36 x 32 x 92
// quadratic (3456) 11786 -> 11612; but 150 x 40 x 32 x 24 (3840) 3037 and 3060,
// 64^3 x 92 quadratic (4096) 14.86 and 15.37 ms.  One wave also where the rows
// just fill the chip once (32 x 44 x 44 x 92, 1936 rows, 3752 and 3778 us; 128
// x 32 x 32 x 92 quadratic, 3072, 10252 and 10612, its moments 2745 and 2871),
// and with few directions, of which four waves have hardly one each, unless the
// rows are very few (moments of 32 x 44 x 44 x 4, 93 and 109 us; 20^3 x 4, 400
// rows, 71 and 63).
static int deposit_slices(const Desc3 &h, bool full)
{
    const bool quad = h.shape == 2;
    const int64_t rows = (int64_t)h.n[1] * h.n[2] * xsegs(h.n[0], quad ? W - 2 : W - 1);
    const int64_t held = 256 * (quad && !full ? 12 : 8);
    if (h.ndir < 8 && 4 * rows > held)
        return 1;
    if (10 * rows > 9 * held && rows <= held)
        return 1;
    return 4 * rows <= 5 * held ? 4 : 1;
}

// workgroups of a deposit launch: patches of rows times x-segments (segments
// of 63 cells for the linear shape, 62 for the quadratic one)
template <int DS>
static unsigned deposit_blocks(const Desc3 &h)
{
    const int sw = (h.shape == 2) ? W - 2 : W - 1;
    return (unsigned)(((h.n[1] + dep_py<DS>() - 1) / dep_py<DS>()) * ((h.n[2] + dep_pz<DS>() - 1) / dep_pz<DS>()) *
                      xsegs(h.n[0], sw));
}

// ---------------------------------------------------------------------------
// Fused linear stages: one kernel per Runge-Kutta stage does the particle
// update and the deposit of the next stage state, plus a small reduction.
//
// A workgroup (FW waves) owns one x-row (y0, z0) of *next-stage* lower
// cells and every direction.  For direction d, lane x takes the particle
// whose lower cell at the next stage time is (x, y0, z0), so all of the
// workgroup's particles deposit into the same four rows (y0 + cy, z0 + cz),
// cy, cz in {0, 1}.  Their current lower cells differ from the next ones by
// delta in {-1, 0, 1} per axis (no particle crosses a whole cell within a
// stage).  The directions are taken class by class (the pair delta_y,
// delta_z; see fclass_at), and the four gather rows (y0 + delta_y + cy,
// z0 + delta_z + cz) of a class are staged in LDS before its directions.
// Row (y0 + dy, z0 + dz), dy and dz in -1 .. 2, goes to LDS slot
// ((dy + 1) & 1) + 2 ((dz + 1) & 1): a class's four rows take four distinct
// slots, and a row that the next class also needs stays where it is, so a
// change of class loads only the rows that change (two, in the class order).
//
// The deposit goes through LDS in rounds of FW directions: every wave
// forms the traceless source X = (N/dV) rho - (Nbar/dV) rhobar^* of its
// direction's next stage state and writes it to its LDS slot; after a
// barrier wave w accumulates source component w of all slots in slot
// order into 16 registers (the 4 destination rows times the groups A, B_x,
// B_y, B_z), pulling cell x's share from particles x (weight 1 - fx) and
// x - 1 (weight fx).  At the end each wave writes its accumulators as the
// partials (slot q = destination row) of its rows, and reduce3f_kernel adds
// the four partials of every cell in slot order: no atomics, bitwise
// reproducible.
// ---------------------------------------------------------------------------
constexpr int FW = 8;
static_assert(NGT % FW == 0, "each wave stages NGT / FW components of a gather row");

__device__ __forceinline__ int near_delta(int d, int n)
{
    // a difference of two shifts mod n that is known to be -1, 0 or 1 (mod n)
    d = (d > 1) ? d - n : d;
    return (d < -1) ? d + n : d;
}

// Directions are taken class by class, a class being the pair (delta_y,
// delta_z) of cell faces crossed in y and z during the stage: first the
// directions that stay in their rows, then each other class, every class in
// ascending direction order.  The four gather rows of a class are staged in
// LDS before its directions, so every gather reads LDS.  The fused kernel
// takes boxes of at most FMAX_DIRS directions.
constexpr int FMAX_DIRS = 1024;

// Value of the lane one below, lane 0 taking lane n - 1 (periodic row of n
// <= 64 cells): DPP wave_shr:1 on the two 32-bit halves, no LDS traffic.
__device__ __forceinline__ double lane_below_wrap(double x, int lane, int n)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x138, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x138, 0xf, 0xf, true);
    const double w = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), n - 1),
                                      __builtin_amdgcn_readlane(__double2loint(x), n - 1));
    return lane == 0 ? w : __hiloint2double(hi, lo);
}

// Value of the lane one above, lane n - 1 taking lane 0: DPP wave_shl:1.
__device__ __forceinline__ double lane_above_wrap(double x, int lane, int n)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x130, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x130, 0xf, 0xf, true);
    const double w = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 0),
                                      __builtin_amdgcn_readlane(__double2loint(x), 0));
    return lane == n - 1 ? w : __hiloint2double(hi, lo);
}

// class index of (delta_y, delta_z) in {-1, 0, 1}^2, and the order in which
// classes are taken: (0, 0) first, then once round the ring, (1, 0), (1, 1),
// (0, 1), (-1, 1), (-1, 0), (-1, -1), (0, -1), (1, -1), so that consecutive
// classes differ by one in delta_y or delta_z and share two gather rows
__device__ __forceinline__ int fclass(int dy, int dz) { return (dy + 1) + 3 * (dz + 1); }
__device__ __forceinline__ int fclass_at(int i) { return (int)((0x210367854ull >> (4 * i)) & 15u); }

// Stage times of a fused linear stage: the current one (gather, update) and
// the next one (deposit).  MODE 5 deposits the current state.
template <int MODE>
__device__ __forceinline__ void fstage_times(int64_t n, double dt, double *t_cur, double *t_next)
{
    if (MODE == 1) {
        *t_cur = stage_time(n, dt, 0.0);
        *t_next = stage_time(n, dt, 0.5);
    } else if (MODE == 2) {
        *t_cur = stage_time(n, dt, 0.5);
        *t_next = *t_cur;
    } else if (MODE == 3) {
        *t_cur = stage_time(n, dt, 0.5);
        *t_next = stage_time(n, dt, 1.0);
    } else if (MODE == 4) {
        *t_cur = stage_time(n, dt, 1.0);
        *t_next = stage_time(n + 1, dt, 0.0);
    } else {
        *t_cur = stage_time(n, dt, 0.0);
        *t_next = *t_cur;
    }
}

// scalar (constant address space) reads of the per-stage tables
typedef const __attribute__((address_space(4))) FDir cFDir;
typedef const __attribute__((address_space(4))) int32_t cint32;

// The stored reals of a slope (no trace entries; see load_slope), and the
// trace entries formed from them afterwards: split so that a kernel can issue
// the loads well before it uses them.
template <bool NT>
__device__ __forceinline__ void load_slope_raw(const double *K, int64_t np, int64_t p, double k[18])
{
#pragma unroll
    for (int c = 1; c < 18; c++)
        if (c != 9)
            k[c] = pld<NT>(K + kslot(c) * np + p);
}

__device__ __forceinline__ void slope_trace(double k[18])
{
    k[0] = -(k[1] + k[2]);
    k[9] = -(k[10] + k[11]);
}

// Row (y0 + dy, z0 + dz) of grid G for a row code (dy + 1) + 4 (dz + 1),
// dy, dz in -1 .. 2 (periodic)
__device__ __forceinline__ const double *row_of(const double *G, unsigned code, int y0, int z0, int nx,
                                                int ny, int nz)
{
    int yy = y0 + (int)(code & 3u) - 1, zz = z0 + (int)(code >> 2) - 1;
    yy = (yy < 0) ? yy + ny : (yy >= ny ? yy - ny : yy);
    yy = (yy >= ny) ? yy - ny : yy;
    zz = (zz < 0) ? zz + nz : (zz >= nz ? zz - nz : zz);
    zz = (zz >= nz) ? zz - nz : zz;
    return G + ((int64_t)zz * ny + yy) * nx;
}

typedef const __attribute__((address_space(4))) Desc3 cDesc3;

// Deposit of one round's sources (slots 0 .. nslot-1 of LDS buffer buf)
// into this wave's accumulators: source component kown of every slot, in
// slot order, pulling cell x's share from particles x and x - 1.
__device__ __forceinline__ void fused_accumulate(const double (*Xb)[FW * W], const double (*Pb)[18],
                                                 int nslot, int kown, int lane, int nx, double acc[16])
{
    for (int j = 0; j < nslot; ++j) {
        const double *ps = Pb[j];
        const double fx = ps[0];
        const double xv = Xb[kown][j * W + lane];
        const double xl = lane_below_wrap(xv, lane, nx);
        const double xc = wsum2(1.0 - fx, xv, fx, xl);
#pragma unroll
        for (int i = 0; i < 16; i++)
            acc[i] += ps[1 + i] * xc;
    }
}

template <int MODE>
__global__ void __launch_bounds__(FW * W)
stage3f_kernel(const Desc3 *__restrict__ dp)
{
    __shared__ double Gt[MODE == 5 ? 1 : 4 * NGT * W];  // [row slot][comp][x]
    __shared__ double Xs[2][NXT][FW * W];                // [buf][source comp][slot][x]
    __shared__ double Ps[2][FW][18];                     // fxn, c[16] of a slot's direction
    // The descriptor is read through the constant address space: its fields
    // are scalar loads that no store of the kernel can alias, so the compiler
    // may load them when used and keep or reload them freely.
    const cDesc3 &S = *(const cDesc3 *)dp;
    const cFDir *ft = (const cFDir *)S.ftab;
    const cint32 *ford = (const cint32 *)S.forder;
    const cint32 *fend = (const cint32 *)S.fcls_end;
    const int lane = threadIdx.x & (W - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / W);
    const int nx = S.n[0], ny = S.n[1], nz = S.n[2];
    const int row = S.rowmap[blockIdx.x];
    const int y0 = row % ny, z0 = row / ny;
    const bool active = lane < nx;
    const double dt = S.dt;
    const double *Gin = S.G[(MODE - 1) & 1];
    const double *Kp = (MODE == 2) ? S.K1 : (MODE == 3) ? S.K2 : S.K3;

    // this wave's share of the deposit: source component k = wave, all four
    // destination rows q and all four groups A, B_x, B_y, B_z
    const int kown = wave;
    double acc[16];
#pragma unroll
    for (int i = 0; i < 16; i++)
        acc[i] = 0.0;

    // A round's deposit is accumulated during the next round, once that
    // round's particle loads are in flight (its own buffers stay untouched
    // until the barrier after that round).
    int round = 0, pend = 0;  // slots of the previous round still to deposit
    unsigned held = ~0u;      // the row held by each LDS slot, 5 bits a slot (31: none)
    for (int ci = 0; ci < 9; ++ci) {
        const int cbeg = (ci == 0) ? 0 : fend[ci - 1], cend = fend[ci];
        if (cbeg == cend)
            continue;  // uniform
        const int c = fclass_at(ci);
        const int dys = c % 3 - 1, dzs = c / 3 - 1;
        // gather row q = 2 qz + qy of the class, (y0 + dys + qy, z0 + dzs +
        // qz), is LDS slot q ^ xm (see the row slots above)
        const int xm = ((dys + 1) & 1) | (((dzs + 1) & 1) << 1);
        if (MODE != 5) {
            // the slots whose row changes (workgroup-uniform)
            int load = 0;
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int sl = q ^ xm;
                const unsigned code = (unsigned)((dys + (q & 1) + 1) + 4 * (dzs + (q >> 1) + 1));
                if (((held >> (5 * sl)) & 31u) != code) {
                    load |= 1 << sl;
                    held = (held & ~(31u << (5 * sl))) | (code << (5 * sl));
                }
            }
            if (load) {
                // the changing rows, two at a time: wave w loads components
                // w, w + FW, w + 2 FW, w + 3 FW of each (one 64-lane row
                // segment per load); the first two are in flight while the
                // waves meet at the barrier after the previous class's
                // gathers, before any LDS store
                int rest = load;
                bool first = round > 0;
                while (rest) {
                    const int sa = __builtin_ctz(rest);
                    rest &= rest - 1;
                    const int sb = rest ? __builtin_ctz(rest) : sa;
                    const bool two = rest != 0;
                    if (two)
                        rest &= rest - 1;
                    double va[NGT / FW], vb[NGT / FW];
                    const double *pa = row_of(Gin, (held >> (5 * sa)) & 31u, y0, z0, nx, ny, nz) + lane;
                    const double *pb = row_of(Gin, (held >> (5 * sb)) & 31u, y0, z0, nx, ny, nz) + lane;
#pragma unroll
                    for (int e = 0; e < NGT / FW; e++) {
                        va[e] = active ? gld(pa + (int64_t)(wave + FW * e) * S.ncell) : 0.0;
                        vb[e] = (active && two) ? gld(pb + (int64_t)(wave + FW * e) * S.ncell) : 0.0;
                    }
                    if (first)
                        __syncthreads();  // the previous class's gathers are done
                    first = false;
#pragma unroll
                    for (int e = 0; e < NGT / FW; e++) {
                        Gt[(sa * NGT + wave + FW * e) * W + lane] = va[e];
                        if (two)
                            Gt[(sb * NGT + wave + FW * e) * W + lane] = vb[e];
                    }
                }
                __syncthreads();
            }
        }
        for (int i0 = cbeg; i0 < cend; i0 += FW, ++round) {
            const int buf = round & 1;
            const int idx = i0 + wave;
            const bool has = idx < cend;  // wave-uniform
            const int d = has ? ford[idx] : 0;
            const cFDir &F = ft[d];
            int64_t p = 0;
            double Y[18], k1[18], k2[18], k3[18];
            double pval = 0.0;
            if (has) {
                // the slot's deposit weights (17 reals, one per lane), loaded
                // before the particle data, stored to LDS after the deposit of
                // the previous round (the store waits for this load only)
                if (lane < 17)
                    pval = gld(reinterpret_cast<const double *>(S.ftab + d) + FDIR_DEP + lane);
                // the particle whose next-stage lower cell is (lane, y0, z0):
                // issue its loads first
                int cx = lane - F.rxn, cy = y0 - F.ryn, cz = z0 - F.rzn;
                cx = (cx < 0) ? cx + nx : cx;
                cy = (cy < 0) ? cy + ny : cy;
                cz = (cz < 0) ? cz + nz : cz;
                const int64_t cc = ((int64_t)cz * ny + cy) * nx + (active ? cx : 0);
                p = (int64_t)d * S.ncell + cc;
                // (lanes past the row load a valid particle, cell 0's, and
                // store nothing)
#pragma unroll
                for (int k = 0; k < 18; k++)
                    Y[k] = fpic::gld_nt(S.Y + k * S.np + p);
                if (MODE == 4) {
                    load_slope_raw<true>(S.K1, S.np, p, k1);
                    load_slope_raw<true>(S.K2, S.np, p, k2);
                    load_slope_raw<true>(S.K3, S.np, p, k3);
                } else if (MODE == 2 || MODE == 3) {
                    load_slope_raw<true>(Kp, S.np, p, k1);
                }
            }
            if (pend)
                fused_accumulate(Xs[buf ^ 1], Ps[buf ^ 1], pend, kown, lane, nx, acc);
            if (has) {
                if (lane < 17)
                    Ps[buf][wave][lane] = pval;
                double yn[18];
                if (MODE == 5) {
#pragma unroll
                    for (int k = 0; k < 18; k++)
                        yn[k] = Y[k];
                } else {
                    double yv[18], base[18];
                    if (MODE == 1) {
#pragma unroll
                        for (int k = 0; k < 18; k++)
                            yv[k] = base[k] = Y[k];
                    } else if (MODE == 4) {
                        const double h6 = dt / 6.0;
                        slope_trace(k1);
                        slope_trace(k2);
                        slope_trace(k3);
#pragma unroll
                        for (int k = 0; k < 18; k++) {
                            yv[k] = Y[k] + dt * k3[k];
                            const double ks = (k1[k] + 2.0 * k2[k]) + 2.0 * k3[k];
                            base[k] = Y[k] + h6 * ks;
                        }
                    } else {
                        const double a = 0.5 * dt;
                        slope_trace(k1);
#pragma unroll
                        for (int k = 0; k < 18; k++) {
                            yv[k] = Y[k] + a * k1[k];
                            base[k] = Y[k];
                        }
                    }
                    // current lower cell = next lower cell + (dxs, dys, dzs):
                    // the four staged rows, then x with the lane to the right
                    int xa = lane + F.dxs;
                    xa = (xa < 0) ? xa + nx : (xa >= nx ? xa - nx : xa);
                    xa = active ? xa : 0;
                    const double fx = F.fx;
                    // the y/z weight of the row in each LDS slot (row q of
                    // the class is in slot q ^ xm); summed in slot order
                    double wsl[4];
#pragma unroll
                    for (int sl = 0; sl < 4; sl++)
                        wsl[sl] = F.wyz[sl ^ xm];
                    double ra[NXT];
#pragma unroll
                    for (int k = 0; k < NXT; k++)
                        ra[k] = 0.0;
#pragma unroll 1
                    for (int grp4 = 0; grp4 < 4; grp4++) {
                        const double coef = (grp4 == 0) ? 1.0 : (grp4 == 1) ? -F.vx : (grp4 == 2) ? -F.vy : -F.vz;
                        const double *g = Gt + NXT * grp4 * W + xa;
#pragma unroll
                        for (int sl = 0; sl < 4; sl++) {
                            const double c = coef * wsl[sl];
#pragma unroll
                            for (int k = 0; k < NXT; k++)
                                ra[k] += c * g[(sl * NGT + k) * W];
                        }
                    }
                    double Hnn[9];
                    Hnn[0] = 0.0;
#pragma unroll
                    for (int k = 0; k < NXT; k++)
                        Hnn[k + 1] = (1.0 - fx) * ra[k] + fx * lane_above_wrap(ra[k], lane, nx);
                    double H[9], Hb[9], kk[18];
#pragma unroll
                    for (int k = 0; k < 9; k++) {
                        H[k] = S.hvac[k] + Hnn[k];
                        const double hb = S.hvacb[k] - Hnn[k];
                        Hb[k] = (k == 4 || k == 6 || k == 8) ? -hb : hb;
                    }
                    commutator(H, yv, kk);
                    commutator(Hb, yv + 9, kk + 9);
                    if (MODE == 4) {
                        const double h6 = dt / 6.0;
#pragma unroll
                        for (int k = 0; k < 18; k++) {
                            yn[k] = base[k] + h6 * kk[k];
                            if (active)
                                fpic::gst_nt(S.Y + k * S.np + p, yn[k]);
                        }
                    } else {
                        double *Ko = (MODE == 1) ? S.K1 : (MODE == 2) ? S.K2 : S.K3;
                        const double an = (MODE == 3) ? dt : 0.5 * dt;
#pragma unroll
                        for (int k = 0; k < 18; k++) {
                            if (active && k != 0 && k != 9)
                                fpic::gst_nt(Ko + kslot(k) * S.np + p, kk[k]);
                            yn[k] = base[k] + an * kk[k];
                        }
                    }
                }
                // the traceless source of the next stage state into this wave's slot
                const double wN = F.wN, wNb = F.wNb;
                double x[9];
#pragma unroll
                for (int k = 0; k < 9; k++)
                    x[k] = source_comp(k, wN, yn[k], wNb, yn[9 + k]);
                double *xs = &Xs[buf][0][wave * W + lane];
                xs[0 * FW * W] = active ? x[1] - x[0] : 0.0;
                xs[1 * FW * W] = active ? x[2] - x[0] : 0.0;
#pragma unroll
                for (int k = 3; k < 9; k++)
                    xs[(k - 1) * FW * W] = active ? x[k] : 0.0;
            }
            __syncthreads();
            pend = min(FW, cend - i0);
        }
    }
    if (pend)
        fused_accumulate(Xs[(round - 1) & 1], Ps[(round - 1) & 1], pend, kown, lane, nx, acc);
    if (active) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            int yy = y0 + (q & 1), zz = z0 + (q >> 1);
            yy = (yy >= ny) ? yy - ny : yy;
            zz = (zz >= nz) ? zz - nz : zz;
            const int64_t cell = ((int64_t)zz * ny + yy) * nx + lane;
            double *P = S.P4 + (int64_t)q * NGT * S.ncell;
#pragma unroll
            for (int g = 0; g < 4; g++)
                gst(P + (int64_t)(NXT * g + kown) * S.ncell + cell, acc[4 * q + g]);
        }
    }
}

// Direction table of fused stage NEXT at step n (threads of one workgroup;
// lcls: LDS scratch of FMAX_DIRS entries).
template <int NEXT>
__device__ void build_dirtab(const Desc3 &S, int64_t n, signed char *lcls)
{
    const int nx = S.n[0], ny = S.n[1], nz = S.n[2];
    double t_cur, t_next;
    fstage_times<NEXT>(n, S.dt, &t_cur, &t_next);
    for (int d = threadIdx.x; d < S.ndir; d += blockDim.x) {
        const double vx = tld(S.v[0], d), vy = tld(S.v[1], d), vz = tld(S.v[2], d);
        int rxn, ryn, rzn, rx, ry, rz;
        double fxn, fyn, fzn, fx, fy, fz;
        axis_shift(vx, t_next, S.dx[0], nx, &rxn, &fxn);
        axis_shift(vy, t_next, S.dx[1], ny, &ryn, &fyn);
        axis_shift(vz, t_next, S.dx[2], nz, &rzn, &fzn);
        axis_shift(vx, t_cur, S.dx[0], nx, &rx, &fx);
        axis_shift(vy, t_cur, S.dx[1], ny, &ry, &fy);
        axis_shift(vz, t_cur, S.dx[2], nz, &rz, &fz);
        FDir F;
        F.rxn = rxn;
        F.ryn = ryn;
        F.rzn = rzn;
        F.dxs = near_delta(rx - rxn, nx);
        F.cls = fclass(near_delta(ry - ryn, ny), near_delta(rz - rzn, nz));
        F.pad_[0] = F.pad_[1] = F.pad_[2] = 0;
        F.fx = fx;
        F.fxn = fxn;
        const double m[4] = {1.0, vx, vy, vz};
#pragma unroll
        for (int qz = 0; qz < 2; qz++)
#pragma unroll
            for (int qy = 0; qy < 2; qy++) {
                const int q = 2 * qz + qy;
                F.wyz[q] = (qy ? fy : 1.0 - fy) * (qz ? fz : 1.0 - fz);
                const double wq = (qy ? fyn : 1.0 - fyn) * (qz ? fzn : 1.0 - fzn);
#pragma unroll
                for (int g = 0; g < 4; g++)
                    F.c[4 * q + g] = wq * m[g];
            }
        F.vx = vx;
        F.vy = vy;
        F.vz = vz;
        F.wN = tld(S.wN, d);
        F.wNb = tld(S.wNb, d);
        F.pad2_[0] = F.pad2_[1] = 0.0;
        S.ftab[d] = F;
        lcls[d] = (signed char)F.cls;
    }
    __syncthreads();
    if (threadIdx.x < W) {
        const int lane = threadIdx.x;
        int at = 0;
        for (int ci = 0; ci < 9; ++ci) {
            const int c = fclass_at(ci);
            for (int d0 = 0; d0 < S.ndir; d0 += W) {
                const int d = d0 + lane;
                const bool take = d < S.ndir && lcls[d] == c;
                const uint64_t mask = __ballot(take);
                if (take)
                    S.forder[at + __popcll(mask & ((1ull << lane) - 1ull))] = d;
                at += __popcll(mask);
            }
            if (lane == 0)
                S.fcls_end[ci] = at;
        }
    }
}

// The direction table and class order of one fused stage (one workgroup).
template <int MODE>
__global__ void __launch_bounds__(1024) dirtab3f_kernel(const Desc3 *__restrict__ dp)
{
    __shared__ signed char lcls[FMAX_DIRS];
    build_dirtab<MODE>(*dp, *dp->step, lcls);
}

// G[out_buf] = the sum of the four partial grids of a fused stage, in slot
// order (traceless components).  Workgroup 0 also writes the direction table
// of the next stage, NEXT, at step n + step_ahead, and then, if tick, moves
// the step counter on by one (the next stage belongs to the next step).
template <int NEXT>
__global__ void __launch_bounds__(256) reduce3f_kernel(const Desc3 *__restrict__ dp, int out_buf,
                                                      int step_ahead, int tick)
{
    __shared__ signed char lcls[FMAX_DIRS];
    const Desc3 &S = *dp;
    const int64_t len = (int64_t)NGT * S.ncell;
    double *G = out_buf ? S.G[1] : S.G[0];
    const double *P = S.P4;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < len; i += stride) {
        const double a = fpic::gld_nt(P + i), b = fpic::gld_nt(P + len + i);
        const double c = fpic::gld_nt(P + 2 * len + i), e = fpic::gld_nt(P + 3 * len + i);
        gst(G + i, ((a + b) + c) + e);
    }
    if (blockIdx.x == 0) {
        const int64_t n = *S.step;
        build_dirtab<NEXT>(S, n + step_ahead, lcls);
        __syncthreads();
        if (tick && threadIdx.x == 0)
            *S.step = n + 1;
    }
}

// ---------------------------------------------------------------------------
// Quadratic (triangular-shaped cloud) shape function, Sec. II.B.1.  Along
// each axis a particle spreads over its nearest cell centre and the two
// neighbours with weights (1/2 - xi)^2 / 2, 3/4 - xi^2, (1/2 + xi)^2 / 2,
// xi = x - x_nearest in [-1/2, 1/2) (each operation rounded once, as the CPU
// reference forms them); a one-cell axis gives (0, 1, 0).  The particle
// kernel's workgroup owns one row of *nearest* cells and stages the nine grid
// rows it interpolates from in LDS, as the 32 traceless moment components
// (nine rows of all 36 would not fit the 160 KB at 64 cells per row).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void axis_quad(double v, double t, double dx, int n, int *r, double w[3])
{
#pragma clang fp contract(off)
    if (n == 1) {
        *r = 0;
        w[0] = 0.0;
        w[1] = 1.0;
        w[2] = 0.0;
        return;
    }
    const double u = (v * t) / dx;
    const double fl = floor(u);
    const double phi = u - fl;
    const int up = phi < 0.5 ? 0 : 1;
    const double xi = up ? phi - 1.0 : phi;
    w[0] = 0.5 * ((0.5 - xi) * (0.5 - xi));
    w[1] = 0.75 - xi * xi;
    w[2] = 0.5 * ((0.5 + xi) * (0.5 + xi));
    const double nd = (double)n;
    const double near = fl + (double)up;
    double q = near - nd * floor(near / nd);
    if (q < 0.0)
        q += nd;
    if (q >= nd)
        q -= nd;
    *r = (int)q;
}

__device__ __forceinline__ int wrap(int i, int n)
{
    i %= n;
    return i < 0 ? i + n : i;
}

// i mod n for -2 n <= i < 2 n
__device__ __forceinline__ int wrap1(int i, int n)
{
    i = i < 0 ? i + n : i;
    i = i < 0 ? i + n : i;
    return i >= n ? i - n : i;
}

// w[b] for a run-time b in 0..2, without indexing a private array
__device__ __forceinline__ double pick3(const double w[3], int b)
{
    return b == 0 ? w[0] : (b == 1 ? w[1] : w[2]);
}

// Directions per gather block: each LDS read of a grid row serves the
// block's directions.  Two for stages 1-3; stage 4 holds three slopes and
// keeps one (more would spill).
template <int MODE>
constexpr int qdb() { return MODE == 4 ? 1 : 2; }

template <int MODE, bool NT>
__global__ void __launch_bounds__(MAX_WAVES3 * W)
particle3q_kernel(const Desc3 *__restrict__ dp, int dpw, int nitems)
{
    __shared__ double Gq[9 * NGT * W];   // [row q][component][x], 144 KiB
    const Desc3 S = *dp;
    const int lane = threadIdx.x & (W - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / W);
    const int nwaves = blockDim.x / W;
    const int item = S.n[0] > W ? xcd_item(blockIdx.x, nitems) : (int)blockIdx.x;
    if (item >= nitems)
        return;
    const int nx = S.n[0], ny = S.n[1], nz = S.n[2];
    const int nseg = xsegs(nx, W - 2);
    const int nrs = ny * nz * nseg;
    const int rs = item % nrs, grp = item / nrs;
    const int row = rs / nseg, seg = rs % nseg;
    const int y0 = row % ny, z0 = row / ny;
    const XRow xw = xrow<1, 1>(nx, seg, lane);
    const bool active = xw.own;
    const int64_t n = *S.step;
    const double dt = S.dt;
    double t_cur = 0.0;
    if (MODE == 2 || MODE == 3)
        t_cur = stage_time(n, dt, 0.5);
    else if (MODE == 4)
        t_cur = stage_time(n, dt, 1.0);
    else
        t_cur = stage_time(n, dt, 0.0);
    const double *Gin = S.G[(MODE - 1) & 1];
    const double *Kp = (MODE == 2) ? S.K1 : (MODE == 3) ? S.K2 : S.K3;
    const int dbeg = (grp * nwaves + wave) * dpw, dend = min(dbeg + dpw, S.ndir);
    const int xl = xw.left, xr = xw.right;
    // Stage the nine grid rows around the nearest row (y0, z0) in LDS, row
    // q = 3 c + b being (y0 + b - 1, z0 + c - 1): the 32 traceless moment
    // components of the stage grid (36 would not fit at 64 cells per row).
    // Column j holds the cell of lane j; columns past a whole row (j >= nx)
    // hold 0.
    const int xbase = (nx <= W) ? 0 : seg * (W - 2) - 1 + nx;
    for (int idx = threadIdx.x; idx < 9 * 4 * W; idx += blockDim.x) {
        const int j = idx % W, t = idx / W;
        const int g4 = t % 4, q = t / 4;  // eight components of one matrix per task
        const int b = q % 3, cc = q / 3;
        double v[NXT];
#pragma unroll
        for (int k = 0; k < NXT; k++)
            v[k] = 0.0;
        if (nx > W || j < nx) {
            const int x = (nx <= W) ? j : (xbase + j) % nx;
            const int64_t cell = ((int64_t)wrap(z0 + cc - 1, nz) * ny + wrap(y0 + b - 1, ny)) * nx + x;
#pragma unroll
            for (int k = 0; k < NXT; k++)
                v[k] = gld(Gin + (int64_t)(NXT * g4 + k) * S.ncell + cell);
        }
#pragma unroll
        for (int k = 0; k < NXT; k++)
            Gq[(q * NGT + NXT * g4 + k) * W + j] = v[k];
    }
    __syncthreads();

    constexpr int QDB = qdb<MODE>();
    for (int d0 = dbeg; d0 < dend; d0 += QDB) {
        // weights of the block's directions (past the end: the last one
        // again, not stored)
        double vb[QDB][3], wxb[QDB][3], wyb[QDB][3], wzb[QDB][3];
        int rxb[QDB], ryb[QDB], rzb[QDB];
#pragma unroll
        for (int j = 0; j < QDB; j++) {
            const int d = min(d0 + j, dend - 1);
            vb[j][0] = tld(S.v[0], d);
            vb[j][1] = tld(S.v[1], d);
            vb[j][2] = tld(S.v[2], d);
            axis_quad(vb[j][0], t_cur, S.dx[0], nx, &rxb[j], wxb[j]);
            axis_quad(vb[j][1], t_cur, S.dx[1], ny, &ryb[j], wyb[j]);
            axis_quad(vb[j][2], t_cur, S.dx[2], nz, &rzb[j], wzb[j]);
        }
        // traceless Hnn = A - v.B: components 1..8 of the packed nine
        // (component 0, the ee entry, is 0).  y/z interpolation row by row
        // from LDS, the four groups with their factors into one sum, each read
        // used by every direction of the block; then x once for the sum.
        double Hb4[QDB][NXT];
#pragma unroll
        for (int j = 0; j < QDB; j++)
#pragma unroll
            for (int k = 0; k < NXT; k++)
                Hb4[j][k] = 0.0;
#pragma unroll 1
        for (int grp4 = 0; grp4 < 4; grp4++) {
            double wyc[QDB][3];
#pragma unroll
            for (int j = 0; j < QDB; j++) {
                const double coef = (grp4 == 0) ? 1.0 : -pick3(vb[j], grp4 - 1);
#pragma unroll
                for (int b = 0; b < 3; b++)
                    wyc[j][b] = coef * wyb[j][b];
            }
#pragma unroll 3
            for (int q = 0; q < 9; q++) {
                const int b = q % 3, cc = q / 3;
                const double *gp = Gq + (q * NGT + NXT * grp4) * W + lane;
                double gv[NXT];
#pragma unroll
                for (int k = 0; k < NXT; k++)
                    gv[k] = gp[k * W];
#pragma unroll
                for (int j = 0; j < QDB; j++) {
                    const double wq = pick3(wyc[j], b) * pick3(wzb[j], cc);
#pragma unroll
                    for (int k = 0; k < NXT; k++)
                        Hb4[j][k] += wq * gv[k];
                }
            }
        }
#pragma unroll
        for (int j = 0; j < QDB; j++)
#pragma unroll
            for (int k = 0; k < NXT; k++) {
                const double r = Hb4[j][k], nl = lane_get(r, xl), nr = lane_get(r, xr);
                Hb4[j][k] = (wxb[j][0] * nl + wxb[j][1] * r) + wxb[j][2] * nr;
            }

#pragma unroll 1
        for (int j = 0; j < QDB; j++) {
            const int d = d0 + j;
            if (d >= dend)
                break;
            const double wN = tld(S.wN, d), wNb = tld(S.wNb, d);
            int rx = rxb[0], ry = ryb[0], rz = rzb[0];
            double Hnn[9];
            Hnn[0] = 0.0;
#pragma unroll
            for (int k = 1; k < 9; k++)
                Hnn[k] = Hb4[0][k - 1];
#pragma unroll
            for (int jj = 1; jj < QDB; jj++) {
                const bool m = j == jj;
                rx = m ? rxb[jj] : rx;
                ry = m ? ryb[jj] : ry;
                rz = m ? rzb[jj] : rz;
#pragma unroll
                for (int k = 1; k < 9; k++)
                    Hnn[k] = m ? Hb4[jj][k - 1] : Hnn[k];
            }
            const int cx = wrap1(xw.x - rx, nx), cy = wrap1(y0 - ry, ny), cz = wrap1(z0 - rz, nz);
            const int64_t c = ((int64_t)cz * ny + cy) * nx + (active ? cx : 0);
            const int64_t p = (int64_t)d * S.ncell + c;
            double Y[18];
#pragma unroll
            for (int k = 0; k < 18; k++)
                Y[k] = active ? pld<NT>(S.Y + k * S.np + p) : 0.0;
            double yv[18], base[18], yn[18];
            if (MODE == 1) {
#pragma unroll
                for (int k = 0; k < 18; k++)
                    yv[k] = base[k] = Y[k];
            } else if (MODE == 4) {
                // slopes one at a time into (k1 + 2 k2) + 2 k3 (fewer live
                // registers than holding all three)
                const double h6 = dt / 6.0;
                double ks[18], kt[18];
                load_slope<NT>(S.K1, S.np, p, active, ks);
                load_slope<NT>(S.K2, S.np, p, active, kt);
#pragma unroll
                for (int k = 0; k < 18; k++)
                    ks[k] = ks[k] + 2.0 * kt[k];
                load_slope<NT>(S.K3, S.np, p, active, kt);
#pragma unroll
                for (int k = 0; k < 18; k++) {
                    yv[k] = Y[k] + dt * kt[k];
                    base[k] = Y[k] + h6 * (ks[k] + 2.0 * kt[k]);
                }
            } else {
                double kp[18];
                load_slope<NT>(Kp, S.np, p, active, kp);
#pragma unroll
                for (int k = 0; k < 18; k++) {
                    yv[k] = Y[k] + 0.5 * dt * kp[k];
                    base[k] = Y[k];
                }
            }
            double H[9], Hb[9], kk[18];
#pragma unroll
            for (int k = 0; k < 9; k++) {
                H[k] = S.hvac[k] + Hnn[k];
                const double hb = S.hvacb[k] - Hnn[k];
                Hb[k] = (k == 4 || k == 6 || k == 8) ? -hb : hb;
            }
            commutator(H, yv, kk);
            commutator(Hb, yv + 9, kk + 9);
            if (MODE == 4) {
                const double h6 = dt / 6.0;
#pragma unroll
                for (int k = 0; k < 18; k++) {
                    yn[k] = base[k] + h6 * kk[k];
                    if (active)
                        pst<NT>(S.Y + k * S.np + p, yn[k]);
                }
            } else {
                double *Ko = (MODE == 1) ? S.K1 : (MODE == 2) ? S.K2 : S.K3;
                const double an = (MODE == 3) ? dt : 0.5 * dt;
#pragma unroll
                for (int k = 0; k < 18; k++) {
                    if (active && k != 0 && k != 9)
                        pst<NT>(Ko + kslot(k) * S.np + p, kk[k]);
                    yn[k] = base[k] + an * kk[k];
                }
            }
            if (active)
                store_source<NT>(S, p, wN, wNb, yn);
        }
    }
}

// Quadratic deposit: destination cell (x, y, z) takes weight
// wx[i] wy[j] wz[k] from the particle whose nearest cell is
// (x - i + 1, y - j + 1, z - k + 1), i, j, k = 0..2: nine source rows in y
// and z, then the lanes one right and one left in x.
template <int NC, int DS>
__global__ void __launch_bounds__(DEP_WAVES * W)
deposit3q_kernel(const Desc3 *__restrict__ dp, int half_steps, int out_buf)
{
    const Desc3 S = *dp;
    const int lane = threadIdx.x & (W - 1);
    const int nx = S.n[0], ny = S.n[1], nz = S.n[2];
    const DepWave dw = dep_wave<DS>(ny, nz, xsegs(nx, W - 2), S.ndir);
    const int y = dw.y, z = dw.z, seg = dw.seg;
    const XRow xw = xrow<1, 1>(nx, seg, lane);
    const bool active = xw.valid;
    const int64_t n0 = *S.step;
    double t;
    if (half_steps == 3)
        t = stage_time(n0 + 1, S.dt, 0.0);
    else
        t = stage_time(n0, S.dt, 0.5 * half_steps);
    const int xl = xw.left, xr = xw.right;
    double acc[4 * NC];
#pragma unroll
    for (int q = 0; q < 4 * NC; q++)
        acc[q] = 0.0;
    for (int d = dw.d0; d < dw.d1; ++d) {
        const double vx = tld(S.v[0], d), vy = tld(S.v[1], d), vz = tld(S.v[2], d);
        int rx, ry, rz;
        double wx[3], wy[3], wz[3];
        axis_quad(vx, t, S.dx[0], nx, &rx, wx);
        axis_quad(vy, t, S.dx[1], ny, &ry, wy);
        axis_quad(vz, t, S.dx[2], nz, &rz, wz);
        // the same for the whole wave: row addresses in scalar registers
        rx = __builtin_amdgcn_readfirstlane(rx);
        ry = __builtin_amdgcn_readfirstlane(ry);
        rz = __builtin_amdgcn_readfirstlane(rz);
        const int xs = wrap1(xw.x - rx, nx);
        const int yb = wrap1(y + 1 - ry, ny), zb = wrap1(z + 1 - rz, nz);
        double Xyz[NC];
#pragma unroll
        for (int k = 0; k < NC; k++)
            Xyz[k] = 0.0;
#pragma unroll 1
        for (int kk = 0; kk < 3; kk++)
#pragma unroll
            for (int j = 0; j < 3; j++) {
                const int yy = wrap1(yb - j, ny), zz = wrap1(zb - kk, nz);
                const double w = wy[j] * wz[kk];
                const double *xp = S.X + (int64_t)d * S.ncell + ((int64_t)zz * ny + yy) * nx + xs;
#pragma unroll
                for (int k = 0; k < NC; k++)
                    Xyz[k] += w * (active ? gld(xp + (int64_t)k * S.np) : 0.0);
            }
#pragma unroll
        for (int k = 0; k < NC; k++) {
            const double right = lane_get(Xyz[k], xr), left = lane_get(Xyz[k], xl);
            const double xc = wsum3(wx[0], right, wx[1], Xyz[k], wx[2], left);
            acc[k] += xc;
            acc[NC + k] += vx * xc;
            acc[2 * NC + k] += vy * xc;
            acc[3 * NC + k] += vz * xc;
        }
    }
    if (!dep_join<DS, 4 * NC>(dw, lane, acc))
        return;
    if (xw.own) {
        double *G = out_buf ? S.G[1] : S.G[0];
        const int64_t cell = ((int64_t)z * ny + y) * nx + xw.x;
#pragma unroll
        for (int q = 0; q < 4 * NC; q++)
            gst(G + (int64_t)q * S.ncell + cell, acc[q]);
    }
}

// moments of neutrinos (which = 0) or antineutrinos (1) at the current step
// time, written to out[36][ncell] (deposits N rho or Nbar rhobar alone)
__global__ void __launch_bounds__(256)
momsrc3d_kernel(const Desc3 *__restrict__ dp, int which)
{
    const Desc3 S = *dp;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < S.np; p += stride) {
        const int d = (int)(p / S.ncell);
        const double w = which ? tld(S.wNb, d) : tld(S.wN, d);
        for (int k = 0; k < 9; k++)
            gst(S.X + k * S.np + p, w * gld(S.Y + (which * 9 + k) * S.np + p));
    }
}

__global__ void set_step3d(const Desc3 *dp, int64_t v)
{
    if (threadIdx.x == 0)
        *dp->step = v;
}

__global__ void tick3d(const Desc3 *dp)
{
    if (threadIdx.x == 0)
        *dp->step += 1;
}

// block (b, k): component k
__global__ void __launch_bounds__(256) totals3d(const Desc3 *dp, double *partial)
{
    const Desc3 &S = *dp;
    __shared__ double sh[256];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int k = blockIdx.y;
    double s = 0.0;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < S.np; p += stride) {
        const int d = (int)(p / S.ncell);
        s += ((k < 9) ? tld(S.Nw, d) : tld(S.Nbw, d)) * S.Y[k * S.np + p];
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h)
            sh[threadIdx.x] += sh[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        partial[(size_t)blockIdx.x * 18 + k] = sh[0];
}

__global__ void __launch_bounds__(256) check3d(const Desc3 *dp, double *partial)
{
    const Desc3 &S = *dp;
    __shared__ double sh[3][256];
    double e0 = 0.0, e1 = 0.0, bad = 0.0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < S.np; p += stride) {
        double v[18];
        for (int k = 0; k < 18; ++k) {
            v[k] = S.Y[k * S.np + p];
            if (!isfinite(v[k]))
                bad += 1.0;
        }
        e0 = fmax(e0, fabs(v[0] + v[1] + v[2] - 1.0));
        e1 = fmax(e1, fabs(v[9] + v[10] + v[11] - 1.0));
    }
    sh[0][threadIdx.x] = e0;
    sh[1][threadIdx.x] = e1;
    sh[2][threadIdx.x] = bad;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            sh[0][threadIdx.x] = fmax(sh[0][threadIdx.x], sh[0][threadIdx.x + h]);
            sh[1][threadIdx.x] = fmax(sh[1][threadIdx.x], sh[1][threadIdx.x + h]);
            sh[2][threadIdx.x] += sh[2][threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int q = 0; q < 3; ++q)
            partial[blockIdx.x * 3 + q] = sh[q][0];
}

__global__ void finish_sums(const double *partial, int nblk, int width, int is_check, double *out)
{
    const int k = threadIdx.x;
    if (k >= width)
        return;
    double s = 0.0;
    // (the sums are one chain, their loads sixteen at a time)
#pragma unroll 16
    for (int b = 0; b < nblk; ++b) {
        const double v = partial[(size_t)b * width + k];
        s = (is_check && k < 2) ? fmax(s, v) : s + v;
    }
    out[k] = s;
}

// ------------------------------------------------------------------ host
#define HIPCHECK(x)                                                                     \
    do {                                                                                \
        hipError_t e_ = (x);                                                            \
        if (e_ != hipSuccess)                                                           \
            return fail(FPIC_EHIP, std::string(#x) + ": " + hipGetErrorString(e_));    \
    } while (0)

constexpr int kBlk = 256;  // blocks of the diagnostic reductions

struct Ctx3D {
    Desc3 h;
    Desc3 *d = nullptr;
    char *ws = nullptr;
    hipStream_t stream = nullptr, cap = nullptr;
    int waves = 8, dpw = 0, ngroup = 0, spg = 8, nitems = 0;
    bool fused = false;  // linear shape: fused stage kernels
    int nrows = 0;
    double *scratch = nullptr, *hbuf = nullptr;
    hipGraphExec_t g1 = nullptr, gK = nullptr;
    bool state_set = false;
};

static size_t al(size_t x) { return (x + 255) & ~size_t(255); }

struct Layout {
    size_t tab, Y, K1, K2, K3, X, G0, G1, P4, rowmap, ftab, forder, fcls, step, desc, scratch, total;
    int waves, dpw, ngroup, spg;
    bool fused;
};

static int validate(const fpic_config &c)
{
    if (c.ncell[0] < 1 || c.ncell[1] < 1 || c.ncell[2] < 1 || c.ndir < 1)
        return fail(FPIC_EINVAL, "cell and direction counts must be >= 1");
    if (!c.dirs || !c.N || !c.Nbar)
        return fail(FPIC_EINVAL, "dirs, N and Nbar must be non-null host arrays");
    if (c.shape_order != 1 && c.shape_order != 2)
        return fail(FPIC_EUNSUPPORTED,
                    "shape_order must be 1 (linear, cloud in cell) or 2 (quadratic)");
    if (!(c.dt > 0.0) || !std::isfinite(c.dt))
        return fail(FPIC_EINVAL, "dt must be positive and finite");
    for (int a = 0; a < 3; ++a)
        if (!(c.dx[a] > 0.0) || !std::isfinite(c.dx[a]))
            return fail(FPIC_EINVAL, "cell widths must be positive and finite");
    if ((int64_t)c.ncell[0] * c.ncell[1] * c.ncell[2] > ((int64_t)1 << 30))
        return fail(FPIC_EINVAL, "too many cells");
    double hmax = 0.0;
    for (int i = 0; i < 18; ++i) {
        if (!std::isfinite(c.hvac[i]))
            return fail(FPIC_EINVAL, "hvac has a non-finite entry");
        hmax = std::max(hmax, std::fabs(c.hvac[i]));
    }
    for (int a = 0; a < 3; ++a)
        if (!std::isfinite(c.vmat[a]))
            return fail(FPIC_EINVAL, "vmat has a non-finite entry");
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            const double re = c.hvac[2 * (3 * i + j)], im = c.hvac[2 * (3 * i + j) + 1];
            const double rt = c.hvac[2 * (3 * j + i)], it = c.hvac[2 * (3 * j + i) + 1];
            if (std::fabs(re - rt) + std::fabs(im + it) > 1e-12 * (1.0 + hmax))
                return fail(FPIC_EINVAL, "hvac is not Hermitian");
        }
    double vmax[3] = {0, 0, 0};
    for (int d = 0; d < c.ndir; ++d) {
        const double *v = c.dirs + 3 * d;
        const double n2 = v[0] * v[0] + v[1] * v[1] + v[2] * v[2];
        if (!std::isfinite(n2) || std::fabs(n2 - 1.0) > 1e-9)
            return fail(FPIC_EINVAL, "directions must be unit vectors");
        if (!std::isfinite(c.N[d]) || !std::isfinite(c.Nbar[d]))
            return fail(FPIC_EINVAL, "weights must be finite");
        for (int a = 0; a < 3; ++a)
            vmax[a] = std::max(vmax[a], std::fabs(v[a]));
    }
    for (int a = 0; a < 3; ++a)
        if (c.ncell[a] > 1 && 0.5 * c.dt * vmax[a] / c.dx[a] >= 1.0 - 1e-9)
            return fail(FPIC_EUNSUPPORTED,
                        "dt too large: a particle may cross a whole cell within one "
                        "Runge-Kutta stage (need dt/2 * max|Omega| < dx)");
    return FPIC_OK;
}

static int layout(const fpic_config &c, const fpic_tuning *t, Layout &L)
{
    int rc = validate(c);
    if (rc)
        return rc;
    const int64_t nc = (int64_t)c.ncell[0] * c.ncell[1] * c.ncell[2];
    const int64_t np = nc * c.ndir;
    // x-rows, or x-segments of rows longer than a wave, of the particle kernels
    const int64_t nrows = (int64_t)c.ncell[1] * c.ncell[2] * xsegs(c.ncell[0], c.shape_order == 2 ? W - 2 : W - 1);
    L.waves = (t && t->waves) ? t->waves : 8;
    if (L.waves != 1 && L.waves != 2 && L.waves != 4 && L.waves != MAX_WAVES3)
        return fail(FPIC_EINVAL, "waves must be 1, 2, 4 or 8 for 3D boxes");
    L.dpw = (t && t->dirs_per_wave) ? t->dirs_per_wave : 0;
    if (L.dpw < 0 || L.dpw > 4096)
        return fail(FPIC_EINVAL, "dirs_per_wave out of range");
    if (!L.dpw) {
        // one direction group per row when there are enough rows to fill
        // the chip (about 2048 workgroups), more groups otherwise
        const int64_t groups = std::max<int64_t>(1, (2048 + nrows - 1) / nrows);
        const int64_t dpg = std::max<int64_t>(L.waves, (c.ndir + groups - 1) / groups);
        L.dpw = (int)((dpg + L.waves - 1) / L.waves);
    }
    const int dpg = L.waves * L.dpw;
    L.ngroup = (c.ndir + dpg - 1) / dpg;
    L.spg = (t && t->steps_per_graph) ? t->steps_per_graph : 8;
    if (L.spg < 1 || L.spg > 256)
        return fail(FPIC_EINVAL, "steps_per_graph must be in 1..256");
    const int fused = t ? t->fused : 0;
    if (fused < 0 || fused > 2)
        return fail(FPIC_EINVAL, "fused must be 0, 1 or 2");
    L.fused = c.shape_order == 1 && fused != 2 && c.ndir <= FMAX_DIRS && c.ncell[0] <= W;
    size_t off = 0;
    auto take = [&](size_t b) {
        off = al(off);
        size_t o = off;
        off += b;
        return o;
    };
    const size_t st = sizeof(double) * 18 * (size_t)np;
    const size_t sk = sizeof(double) * fpic::NK * (size_t)np;
    L.tab = take(sizeof(double) * 7 * c.ndir);
    L.Y = take(st);
    L.K1 = take(sk);
    L.K2 = take(sk);
    L.K3 = take(sk);
    L.X = take(sizeof(double) * 9 * (size_t)np);
    L.G0 = take(sizeof(double) * NG * (size_t)nc);
    L.G1 = take(sizeof(double) * NG * (size_t)nc);
    L.P4 = take(L.fused ? sizeof(double) * 4 * NGT * (size_t)nc : 0);
    L.rowmap = take(sizeof(int32_t) * (size_t)nrows);
    L.ftab = take(L.fused ? sizeof(FDir) * (size_t)c.ndir : 0);
    L.forder = take(L.fused ? sizeof(int32_t) * (size_t)c.ndir : 0);
    L.fcls = take(sizeof(int32_t) * 9);
    L.step = take(sizeof(int64_t));
    L.desc = take(sizeof(Desc3));
    L.scratch = take(sizeof(double) * (18 + 18 * kBlk + 3 * kBlk + 3));
    L.total = al(off);
    return FPIC_OK;
}

int workspace_bytes(const fpic_config &cfg, const fpic_tuning *tune, size_t *bytes)
{
    Layout L;
    int rc = layout(cfg, tune, L);
    if (rc)
        return rc;
    *bytes = L.total;
    return FPIC_OK;
}

// stage `mode` (1..4; 5 = deposit sources of the current state) of the
// particle kernels, and the deposit of the sources, for the box's shape order
template <bool NT>
static void launch_particle_nt(const Ctx3D *c, int mode, hipStream_t s)
{
    // MODE 5 is the linear kernel in both shapes: its own x-segments
    const int items5 = c->h.n[1] * c->h.n[2] * xsegs(c->h.n[0], W - 1) * c->ngroup;
    const dim3 pgrid(mode == 5 ? items5 : c->nitems), pblk(c->waves * W);
    const bool q = c->h.shape == 2;
    switch (mode) {
    case 1:
        if (q) particle3q_kernel<1, NT><<<pgrid, pblk, 0, s>>>(c->d, c->dpw, c->nitems);
        else particle3d_kernel<1, NT><<<pgrid, pblk, 0, s>>>(c->d, c->dpw, c->nitems);
        break;
    case 2:
        if (q) particle3q_kernel<2, NT><<<pgrid, pblk, 0, s>>>(c->d, c->dpw, c->nitems);
        else particle3d_kernel<2, NT><<<pgrid, pblk, 0, s>>>(c->d, c->dpw, c->nitems);
        break;
    case 3:
        if (q) particle3q_kernel<3, NT><<<pgrid, pblk, 0, s>>>(c->d, c->dpw, c->nitems);
        else particle3d_kernel<3, NT><<<pgrid, pblk, 0, s>>>(c->d, c->dpw, c->nitems);
        break;
    case 4:
        if (q) particle3q_kernel<4, NT><<<pgrid, pblk, 0, s>>>(c->d, c->dpw, c->nitems);
        else particle3d_kernel<4, NT><<<pgrid, pblk, 0, s>>>(c->d, c->dpw, c->nitems);
        break;
    default:  // no interpolation: the same for both shapes
        particle3d_kernel<5, NT><<<pgrid, pblk, 0, s>>>(c->d, c->dpw, items5);
        break;
    }
}

static void launch_particle(const Ctx3D *c, int mode, hipStream_t s)
{
    if (streams(c->h))
        launch_particle_nt<true>(c, mode, s);
    else
        launch_particle_nt<false>(c, mode, s);
}

template <int DS>
static void launch_deposit_ds(const Ctx3D *c, const Desc3 *dd, int half_steps, int out_buf, hipStream_t s, bool full)
{
    const dim3 dgrid(deposit_blocks<DS>(c->h)), blk(DEP_WAVES * W);
    if (c->h.shape == 2) {
        if (full)
            deposit3q_kernel<9, DS><<<dgrid, blk, 0, s>>>(dd, half_steps, out_buf);
        else
            deposit3q_kernel<NXT, DS><<<dgrid, blk, 0, s>>>(dd, half_steps, out_buf);
    } else {
        if (full)
            deposit3d_kernel<9, DS><<<dgrid, blk, 0, s>>>(dd, half_steps, out_buf);
        else
            deposit3d_kernel<NXT, DS><<<dgrid, blk, 0, s>>>(dd, half_steps, out_buf);
    }
}

// The stage deposits (traceless sources, NGT grid components); full = true
// for the moments diagnostic (all nine source components, 36 per cell).
static void launch_deposit(const Ctx3D *c, const Desc3 *dd, int half_steps, int out_buf, hipStream_t s,
                           bool full = false)
{
    if (deposit_slices(c->h, full) == 4)
        launch_deposit_ds<4>(c, dd, half_steps, out_buf, s, full);
    else
        launch_deposit_ds<1>(c, dd, half_steps, out_buf, s, full);
}

// fused linear stage `mode` (1..4; 5 = deposit of the current state) and
// the reduction of its partials into G[out_buf]
// The direction table of fused linear stage `mode` (1..4; 5 = deposit of
// the current state), and the stage kernel itself.
static void launch_dirtab(const Ctx3D *c, int mode, hipStream_t s)
{
    const dim3 tblk(1024);
    switch (mode) {
    case 1: dirtab3f_kernel<1><<<1, tblk, 0, s>>>(c->d); break;
    case 2: dirtab3f_kernel<2><<<1, tblk, 0, s>>>(c->d); break;
    case 3: dirtab3f_kernel<3><<<1, tblk, 0, s>>>(c->d); break;
    case 4: dirtab3f_kernel<4><<<1, tblk, 0, s>>>(c->d); break;
    default: dirtab3f_kernel<5><<<1, tblk, 0, s>>>(c->d); break;
    }
}

static void launch_stage3f(const Ctx3D *c, int mode, hipStream_t s)
{
    const dim3 grid(c->nrows), blk(FW * W);
    switch (mode) {
    case 1: stage3f_kernel<1><<<grid, blk, 0, s>>>(c->d); break;
    case 2: stage3f_kernel<2><<<grid, blk, 0, s>>>(c->d); break;
    case 3: stage3f_kernel<3><<<grid, blk, 0, s>>>(c->d); break;
    case 4: stage3f_kernel<4><<<grid, blk, 0, s>>>(c->d); break;
    default: stage3f_kernel<5><<<grid, blk, 0, s>>>(c->d); break;
    }
}

// The reduction after fused stage `done` (1..4; 5 = the deposit of the
// current state) into G[out_buf], with the direction table of the stage
// after it; after stage 4 it also moves the step counter on.
static void launch_reduce3f(const Ctx3D *c, int done, hipStream_t s)
{
    const int64_t len = (int64_t)NGT * c->h.ncell;
    const unsigned blocks = (unsigned)std::max<int64_t>(1, std::min<int64_t>(8192, (len + 255) / 256));
    switch (done) {
    case 1: reduce3f_kernel<2><<<blocks, 256, 0, s>>>(c->d, 1, 0, 0); break;
    case 2: reduce3f_kernel<3><<<blocks, 256, 0, s>>>(c->d, 0, 0, 0); break;
    case 3: reduce3f_kernel<4><<<blocks, 256, 0, s>>>(c->d, 1, 0, 0); break;
    case 4: reduce3f_kernel<1><<<blocks, 256, 0, s>>>(c->d, 0, 1, 1); break;
    default: reduce3f_kernel<1><<<blocks, 256, 0, s>>>(c->d, 0, 0, 0); break;
    }
}

// Fused path: deposit the current state (its grid G[0]) and the table of
// stage 1.
static void deposit_current_fused(const Ctx3D *c, hipStream_t s)
{
    launch_dirtab(c, 5, s);
    launch_stage3f(c, 5, s);
    launch_reduce3f(c, 5, s);
}

static hipError_t launch_step(Ctx3D *c, hipStream_t s)
{
    if (c->fused) {
        // stage k reads G[(k-1)&1]; its reduction writes G[k&1] and the
        // table of the next stage (after stage 4: of the next step's first
        // stage, and then moves the step counter on)
        for (int k = 1; k <= 4; ++k) {
            launch_stage3f(c, k, s);
            launch_reduce3f(c, k, s);
        }
        return hipGetLastError();
    }
    // stage s reads G[(s-1)&1]; its deposit writes G[s&1]
    launch_particle(c, 1, s);
    launch_deposit(c, c->d, 1, 1, s);
    launch_particle(c, 2, s);
    launch_deposit(c, c->d, 1, 0, s);
    launch_particle(c, 3, s);
    launch_deposit(c, c->d, 2, 1, s);
    launch_particle(c, 4, s);
    launch_deposit(c, c->d, 3, 0, s);
    tick3d<<<1, 64, 0, s>>>(c->d);
    return hipGetLastError();
}

static int capture(Ctx3D *c, int nsteps, hipGraphExec_t *exec)
{
    HIPCHECK(hipStreamBeginCapture(c->cap, hipStreamCaptureModeThreadLocal));
    hipError_t err = hipSuccess;
    for (int i = 0; i < nsteps && err == hipSuccess; ++i)
        err = launch_step(c, c->cap);
    hipGraph_t g = nullptr;
    hipError_t e2 = hipStreamEndCapture(c->cap, &g);
    if (err != hipSuccess) {
        if (g)
            (void)hipGraphDestroy(g);
        return fail(FPIC_EHIP, std::string("launch during capture: ") + hipGetErrorString(err));
    }
    HIPCHECK(e2);
    hipError_t e3 = hipGraphInstantiate(exec, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    HIPCHECK(e3);
    return FPIC_OK;
}

int create(const fpic_config &cfg, const fpic_tuning *tune, void *ws, size_t bytes, fpic_stream stream,
           Ctx3D **out)
{
    Layout L;
    int rc = layout(cfg, tune, L);
    if (rc)
        return rc;
    if (!ws || bytes < L.total || reinterpret_cast<uintptr_t>(ws) % 256)
        return fail(FPIC_EINVAL, "workspace missing, too small or misaligned");
    Ctx3D *c = new Ctx3D();
    c->ws = static_cast<char *>(ws);
    c->stream = static_cast<hipStream_t>(stream);
    c->waves = L.waves;
    c->dpw = L.dpw;
    c->ngroup = L.ngroup;
    c->spg = L.spg;
    c->nitems = cfg.ncell[1] * cfg.ncell[2] * xsegs(cfg.ncell[0], cfg.shape_order == 2 ? W - 2 : W - 1) *
                L.ngroup;
    c->fused = L.fused;
    c->nrows = cfg.ncell[1] * cfg.ncell[2];
    const int nd = cfg.ndir;
    const double dV = cfg.dx[0] * cfg.dx[1] * cfg.dx[2];
    std::vector<double> tab(7 * (size_t)nd);
    for (int d = 0; d < nd; ++d) {
        for (int a = 0; a < 3; ++a)
            tab[a * nd + d] = cfg.dirs[3 * d + a];
        tab[3 * nd + d] = cfg.N[d] / dV;
        tab[4 * nd + d] = cfg.Nbar[d] / dV;
        tab[5 * nd + d] = cfg.N[d];
        tab[6 * nd + d] = cfg.Nbar[d];
    }
    Desc3 &D = c->h;
    std::memset(&D, 0, sizeof D);
    for (int a = 0; a < 3; ++a) {
        D.n[a] = cfg.ncell[a];
        D.dx[a] = cfg.dx[a];
    }
    D.ndir = nd;
    D.ncell = (int64_t)cfg.ncell[0] * cfg.ncell[1] * cfg.ncell[2];
    D.np = D.ncell * nd;
    D.dt = cfg.dt;
    D.shape = cfg.shape_order;
    const double *h = cfg.hvac;
    const double hv[9] = {h[0], h[8], h[16], h[2], h[3], h[4], h[5], h[10], h[11]};
    for (int k = 0; k < 9; ++k) {
        D.hvac[k] = hv[k] + (k < 3 ? cfg.vmat[k] : 0.0);
        D.hvacb[k] = hv[k] - (k < 3 ? cfg.vmat[k] : 0.0);
    }
    const double *tb = reinterpret_cast<const double *>(c->ws + L.tab);
    for (int a = 0; a < 3; ++a)
        D.v[a] = tb + a * nd;
    D.wN = tb + 3 * nd;
    D.wNb = tb + 4 * nd;
    D.Nw = tb + 5 * nd;
    D.Nbw = tb + 6 * nd;
    D.Y = reinterpret_cast<double *>(c->ws + L.Y);
    D.K1 = reinterpret_cast<double *>(c->ws + L.K1);
    D.K2 = reinterpret_cast<double *>(c->ws + L.K2);
    D.K3 = reinterpret_cast<double *>(c->ws + L.K3);
    D.X = reinterpret_cast<double *>(c->ws + L.X);
    D.G[0] = reinterpret_cast<double *>(c->ws + L.G0);
    D.G[1] = reinterpret_cast<double *>(c->ws + L.G1);
    D.step = reinterpret_cast<int64_t *>(c->ws + L.step);
    D.P4 = L.fused ? reinterpret_cast<double *>(c->ws + L.P4) : nullptr;
    D.rowmap = reinterpret_cast<const int32_t *>(c->ws + L.rowmap);
    D.ftab = L.fused ? reinterpret_cast<FDir *>(c->ws + L.ftab) : nullptr;
    D.forder = L.fused ? reinterpret_cast<int32_t *>(c->ws + L.forder) : nullptr;
    D.fcls_end = reinterpret_cast<int32_t *>(c->ws + L.fcls);
    c->d = reinterpret_cast<Desc3 *>(c->ws + L.desc);
    // The dispatcher hands workgroup b to XCD b % 8, each with its own L2:
    // give every XCD one contiguous run of rows, so that the rows a fused
    // workgroup stages and the partial rows it writes are shared in one L2.
    std::vector<int32_t> rowmap(c->nrows);
    {
        constexpr int kXcds = 8;
        const int n = c->nrows, per = n / kXcds, extra = n % kXcds;
        int start[kXcds], count[kXcds], used[kXcds] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int x = 0, at = 0; x < kXcds; ++x) {
            count[x] = per + (x < extra ? 1 : 0);
            start[x] = at;
            at += count[x];
        }
        for (int b = 0; b < n; ++b) {
            int x = b % kXcds;
            for (int tries = 0; tries < kXcds && used[x] >= count[x]; ++tries)
                x = (x + 1) % kXcds;
            rowmap[b] = start[x] + used[x]++;
        }
    }
    c->scratch = reinterpret_cast<double *>(c->ws + L.scratch);
    hipError_t e = hipMemcpy(c->ws + L.tab, tab.data(), sizeof(double) * tab.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess)
        e = hipMemcpy(c->ws + L.rowmap, rowmap.data(), sizeof(int32_t) * rowmap.size(),
                      hipMemcpyHostToDevice);
    if (e == hipSuccess)
        e = hipMemcpy(c->d, &D, sizeof D, hipMemcpyHostToDevice);
    if (e == hipSuccess)
        e = hipHostMalloc(reinterpret_cast<void **>(&c->hbuf), sizeof(double) * 64, hipHostMallocDefault);
    if (e == hipSuccess)
        e = hipStreamCreateWithFlags(&c->cap, hipStreamNonBlocking);
    if (e != hipSuccess) {
        destroy(c);
        return fail(FPIC_EHIP, std::string("create: ") + hipGetErrorString(e));
    }
    rc = capture(c, 1, &c->g1);
    if (!rc && c->spg > 1)
        rc = capture(c, c->spg, &c->gK);
    if (rc) {
        destroy(c);
        return rc;
    }
    *out = c;
    return FPIC_OK;
}

int set_state(Ctx3D *c, const double *state, int64_t step0)
{
    if (!c || !state)
        return fail(FPIC_EINVAL, "set_state: null argument");
    HIPCHECK(hipMemcpyAsync(c->h.Y, state, sizeof(double) * 18 * c->h.np, hipMemcpyDeviceToDevice, c->stream));
    set_step3d<<<1, 64, 0, c->stream>>>(c->d, step0);
    HIPCHECK(hipGetLastError());
    if (c->fused) {
        deposit_current_fused(c, c->stream);
    } else {
        launch_particle(c, 5, c->stream);
        launch_deposit(c, c->d, 0, 0, c->stream);
    }
    HIPCHECK(hipGetLastError());
    c->state_set = true;
    return FPIC_OK;
}

int get_state(Ctx3D *c, double *state)
{
    if (!c || !state)
        return fail(FPIC_EINVAL, "get_state: null argument");
    HIPCHECK(hipMemcpyAsync(state, c->h.Y, sizeof(double) * 18 * c->h.np, hipMemcpyDeviceToDevice, c->stream));
    return FPIC_OK;
}

int step(Ctx3D *c, int64_t nsteps)
{
    if (!c || nsteps < 0)
        return fail(FPIC_EINVAL, "step: bad argument");
    if (!c->state_set)
        return fail(FPIC_ESTATE, "step before set_state");
    int64_t left = nsteps;
    while (c->spg > 1 && left >= c->spg) {
        HIPCHECK(hipGraphLaunch(c->gK, c->stream));
        left -= c->spg;
    }
    while (left-- > 0)
        HIPCHECK(hipGraphLaunch(c->g1, c->stream));
    return FPIC_OK;
}

int moments(Ctx3D *c, double *out)
{
    if (!c || !out)
        return fail(FPIC_EINVAL, "moments: null argument");
    if (!c->state_set)
        return fail(FPIC_ESTATE, "moments before set_state");
    // the deposit kernel writes G[out_buf]; point a copy of the descriptor
    // at the caller's buffer
    Desc3 D = c->h;
    for (int which = 0; which < 2; ++which) {
        D.G[0] = out + (size_t)which * NG * c->h.ncell;
        HIPCHECK(hipMemcpyAsync(c->scratch, &D, sizeof D, hipMemcpyHostToDevice, c->stream));
        const Desc3 *dd = reinterpret_cast<const Desc3 *>(c->scratch);
        momsrc3d_kernel<<<1024, 256, 0, c->stream>>>(dd, which);
        launch_deposit(c, dd, 0, 0, c->stream, true);
        HIPCHECK(hipGetLastError());
        HIPCHECK(hipStreamSynchronize(c->stream));   // D is a host temporary
    }
    // (the stage kernels rewrite the deposit sources before every deposit)
    return FPIC_OK;
}

int flavor_totals(Ctx3D *c, double *out)
{
    if (!c || !out)
        return fail(FPIC_EINVAL, "flavor_totals: null argument");
    if (!c->state_set)
        return fail(FPIC_ESTATE, "flavor_totals before set_state");
    double *part = c->scratch + 18;
    totals3d<<<dim3(kBlk, 18), 256, 0, c->stream>>>(c->d, part);
    finish_sums<<<1, 64, 0, c->stream>>>(part, kBlk, 18, 0, c->scratch);
    HIPCHECK(hipGetLastError());
    HIPCHECK(hipMemcpyAsync(c->hbuf, c->scratch, sizeof(double) * 18, hipMemcpyDeviceToHost, c->stream));
    HIPCHECK(hipStreamSynchronize(c->stream));
    std::memcpy(out, c->hbuf, sizeof(double) * 18);
    return FPIC_OK;
}

int check(Ctx3D *c, double r[3])
{
    if (!c->state_set)
        return fail(FPIC_ESTATE, "check before set_state");
    double *part = c->scratch + 18 + 18 * kBlk;
    check3d<<<kBlk, 256, 0, c->stream>>>(c->d, part);
    finish_sums<<<1, 64, 0, c->stream>>>(part, kBlk, 3, 1, c->scratch);
    HIPCHECK(hipGetLastError());
    HIPCHECK(hipMemcpyAsync(c->hbuf, c->scratch, sizeof(double) * 3, hipMemcpyDeviceToHost, c->stream));
    HIPCHECK(hipStreamSynchronize(c->stream));
    std::memcpy(r, c->hbuf, sizeof(double) * 3);
    return FPIC_OK;
}

int get_step(Ctx3D *c, int64_t *s)
{
    HIPCHECK(hipMemcpyAsync(c->hbuf, c->h.step, sizeof(int64_t), hipMemcpyDeviceToHost, c->stream));
    HIPCHECK(hipStreamSynchronize(c->stream));
    std::memcpy(s, c->hbuf, sizeof(int64_t));
    return FPIC_OK;
}

int sync(Ctx3D *c)
{
    HIPCHECK(hipStreamSynchronize(c->stream));
    return FPIC_OK;
}

int profile(Ctx3D *c, int nsteps, double *ms)
{
    if (!c->state_set)
        return fail(FPIC_ESTATE, "profile before set_state");
    hipEvent_t ev[9];
    for (auto &e : ev)
        HIPCHECK(hipEventCreate(&e));
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    hipStream_t s = c->stream;
    int rc = FPIC_OK;
    for (int n = 0; n < nsteps && !rc && c->fused; ++n) {
        // per stage: the stage kernel, then its reduction (with the next
        // stage's direction table)
        hipError_t err = hipEventRecord(ev[0], s);
        for (int k = 1; k <= 4 && err == hipSuccess; ++k) {
            launch_stage3f(c, k, s);
            err = hipEventRecord(ev[2 * k - 1], s);
            launch_reduce3f(c, k, s);
            if (err == hipSuccess)
                err = hipEventRecord(ev[2 * k], s);
        }
        if (err == hipSuccess)
            err = hipGetLastError();
        if (err == hipSuccess)
            err = hipEventSynchronize(ev[8]);
        for (int k = 0; k < 8 && err == hipSuccess; ++k) {
            float t = 0.f;
            err = hipEventElapsedTime(&t, ev[k], ev[k + 1]);
            acc[k] += t;
        }
        if (err != hipSuccess)
            rc = fail(FPIC_EHIP, std::string("profile: ") + hipGetErrorString(err));
    }
    for (int n = 0; n < nsteps && !rc && !c->fused; ++n) {
        (void)hipEventRecord(ev[0], s);
        launch_particle(c, 1, s);
        (void)hipEventRecord(ev[1], s);
        launch_deposit(c, c->d, 1, 1, s);
        (void)hipEventRecord(ev[2], s);
        launch_particle(c, 2, s);
        (void)hipEventRecord(ev[3], s);
        launch_deposit(c, c->d, 1, 0, s);
        (void)hipEventRecord(ev[4], s);
        launch_particle(c, 3, s);
        (void)hipEventRecord(ev[5], s);
        launch_deposit(c, c->d, 2, 1, s);
        (void)hipEventRecord(ev[6], s);
        launch_particle(c, 4, s);
        (void)hipEventRecord(ev[7], s);
        launch_deposit(c, c->d, 3, 0, s);
        tick3d<<<1, 64, 0, s>>>(c->d);
        (void)hipEventRecord(ev[8], s);
        hipError_t err = hipGetLastError();
        if (err == hipSuccess)
            err = hipEventSynchronize(ev[8]);
        for (int k = 0; k < 8 && err == hipSuccess; ++k) {
            float t = 0.f;
            err = hipEventElapsedTime(&t, ev[k], ev[k + 1]);
            acc[k] += t;
        }
        if (err != hipSuccess)
            rc = fail(FPIC_EHIP, std::string("profile: ") + hipGetErrorString(err));
    }
    for (auto &e : ev)
        (void)hipEventDestroy(e);
    for (int k = 0; k < 8; ++k)
        ms[k] = acc[k] / nsteps;
    return rc;
}

void diag_buffers(Ctx3D *c, void **stream, double **scratch, double **hbuf, int64_t *ncell)
{
    *stream = c->stream;
    *scratch = c->scratch;
    *hbuf = c->hbuf;
    *ncell = c->h.ncell;
}

void destroy(Ctx3D *c)
{
    if (!c)
        return;
    if (c->stream)
        (void)hipStreamSynchronize(c->stream);
    if (c->g1)
        (void)hipGraphExecDestroy(c->g1);
    if (c->gK)
        (void)hipGraphExecDestroy(c->gK);
    if (c->cap)
        (void)hipStreamDestroy(c->cap);
    if (c->hbuf)
        (void)hipHostFree(c->hbuf);
    delete c;
}

int autotune(const fpic_config &cfg, void *ws, size_t bytes, fpic_stream stream, fpic_tuning *best,
             double *ms_per_step)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    double best_ms = 1e300;
    fpic_tuning bt{};
    int tried = 0;
    std::vector<fpic_tuning> cands;
    if (cfg.shape_order == 1)
        cands.push_back(fpic_tuning{0, 0, 4, 0, 1});  // fused stages
    for (int waves : {2, 4, 8})
        for (int groups : {1, 2, 4}) {
            const int dpw = (cfg.ndir + waves * groups - 1) / (waves * groups);
            if (dpw >= 1 && (groups == 1 || dpw > 1))
                cands.push_back(fpic_tuning{waves, dpw, 4, 0, 2});
        }
    for (const fpic_tuning &t : cands) {
        Ctx3D *c = nullptr;
        int rc = create(cfg, &t, ws, bytes, stream, &c);
        if (rc)
            return rc;
        // any finite state times the same: zeros (deposited as by set_state,
        // which also writes the fused path's first direction table)
        HIPCHECK(hipMemsetAsync(c->h.Y, 0, sizeof(double) * 18 * c->h.np, s));
        set_step3d<<<1, 64, 0, s>>>(c->d, 0);
        if (c->fused)
            deposit_current_fused(c, s);
        else {
            launch_particle(c, 5, s);
            launch_deposit(c, c->d, 0, 0, s);
        }
        HIPCHECK(hipGetLastError());
        c->state_set = true;
        rc = step(c, 2);
        hipEvent_t e0, e1;
        (void)hipEventCreate(&e0);
        (void)hipEventCreate(&e1);
        (void)hipEventRecord(e0, s);
        if (!rc)
            rc = step(c, 4);
        (void)hipEventRecord(e1, s);
        hipError_t es = hipEventSynchronize(e1);
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, e0, e1);
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        destroy(c);
        if (rc)
            return rc;
        if (es != hipSuccess)
            return fail(FPIC_EHIP, hipGetErrorString(es));
        ++tried;
        if (ms / 4 < best_ms) {
            best_ms = ms / 4;
            bt = t;
        }
    }
    if (!tried)
        return fail(FPIC_EINVAL, "no candidate launch shape");
    *best = bt;
    if (ms_per_step)
        *ms_per_step = best_ms;
    return FPIC_OK;
}

}  // namespace fpic3d
