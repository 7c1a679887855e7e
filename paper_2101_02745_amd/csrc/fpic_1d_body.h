// Device code shared by the 1D kernels (fpic_1d.hip: one launch per stage;
// fpic_1d_steps.h: whole steps in one launch): positions, lane moves, the
// slope path, the deposit of one direction and the sums over a workgroup's
// waves and over the direction groups.  The arithmetic stands here once, so
// that both forms round alike, bit for bit.
#pragma once

#include "fpic_device.h"
#include "fpic_internal.h"

namespace fpic {

// Loads and stores of data that other workgroups of the same launch write or
// read (COH): device-coherent 8-byte accesses, past the L2 of the XCD, where
// COH is false ordinary ones.
template <bool COH>
__device__ __forceinline__ double xld(const double *p)
{
    if (COH)
        return __hip_atomic_load((const gdouble *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return gld(p);
}
template <bool COH>
__device__ __forceinline__ void xst(double *p, double v)
{
    if (COH)
        __hip_atomic_store((gdouble *)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        gst(p, v);
}

struct Shift {
    int64_t i;
    double phi;
};

__device__ __forceinline__ Shift shift_of(double v, double t, double dx)
{
#pragma clang fp contract(off)
    const double u = (v * t) / dx;
    const double fl = floor(u);
    Shift s;
    s.i = (int64_t)fl;
    s.phi = u - fl;
    return s;
}

// Value of the lane one below (lane 0 receives 0): DPP wave_shr:1 on the two
// 32-bit halves, no LDS traffic.
__device__ __forceinline__ double lane_below(double x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x138, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x138, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// Value of the lane one above (lane 63 receives 0): DPP wave_shl:1.
__device__ __forceinline__ double lane_above(double x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x130, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x130, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ int pmod_i64(int64_t a, int n)
{
    int64_t r = a % n;
    return (int)(r < 0 ? r + n : r);
}

// r = i mod n for an integer-valued double i (|i| < 2^52), without 64-bit
// integer division.
__device__ __forceinline__ int pmod_dbl(double i, int n)
{
    const double nd = (double)n;
    double r = i - nd * floor(i / nd);
    if (r < 0.0)
        r += nd;
    if (r >= nd)
        r -= nd;
    return (int)r;
}

// The slope path of the 1D stages (gather, Hamiltonians, commutators) is
// written with explicit fused multiply-adds and no other contraction, so a
// slope formed again in a later stage rounds exactly as where it was first
// formed, whatever the surrounding code lets the compiler fuse.

// Neutrino self-interaction part of H at a particle (eq. potentials,
// interpolated with eq. pic_interpolation): the four staged moment groups
// n - nbar^*, f_x, f_y, f_z - fbar^* of the tile Gt (stride gts per
// component) at column kl and fraction phi, combined as n - v.f.
template <int SH>
__device__ __forceinline__ void gather_hnn(const double *Gt, int gts, int kl, double phi, double vx,
                                           double vy, double vz, double Hnn[9])
{
#pragma clang fp contract(off)
    if (SH == 2) {
        const Quad q = quad_weights(phi);
#pragma unroll
        for (int k = 0; k < 9; k++) {
            const double *g = Gt + k * gts + kl - 1 + q.up;
            double B[4];
#pragma unroll
            for (int c = 0; c < 4; c++) {
                const double *h = g + 9 * c * gts;
                B[c] = __builtin_fma(q.w2, h[2], __builtin_fma(q.w1, h[1], q.w0 * h[0]));
            }
            Hnn[k] = __builtin_fma(-vz, B[3], __builtin_fma(-vy, B[2], __builtin_fma(-vx, B[1], B[0])));
        }
    } else {
        const double omp = 1.0 - phi;
#pragma unroll
        for (int k = 0; k < 9; k++) {
            const double *g = Gt + k * gts + kl;
            double B[4];
#pragma unroll
            for (int c = 0; c < 4; c++) {
                const double *h = g + 9 * c * gts;
                B[c] = __builtin_fma(phi, h[1], omp * h[0]);
            }
            Hnn[k] = __builtin_fma(-vz, B[3], __builtin_fma(-vy, B[2], __builtin_fma(-vx, B[1], B[0])));
        }
    }
}

// -i [H, rho] for Hermitian H and rho packed as 9 reals (diagonal, then
// Re/Im of the (0,1), (0,2), (1,2) entries), the same packing and slope as
// commutator() of the shared helpers, each sum of products written as one
// chain of fused multiply-adds.
__device__ __forceinline__ void commutator_fma(const double h[9], const double r[9], double k[9])
{
#pragma clang fp contract(off)
    const double h0 = h[0], h1 = h[1], h2 = h[2];
    const double ar = h[3], ai = h[4], br = h[5], bi = h[6], cr = h[7], ci = h[8];
    const double p0 = r[0], p1 = r[1], p2 = r[2];
    const double xr = r[3], xi = r[4], yr = r[5], yi = r[6], zr = r[7], zi = r[8];
    const double k1 = 2.0 * (__builtin_fma(ar, xi, -(ai * xr)) + __builtin_fma(ci, zr, -(cr * zi)));
    const double k2 = 2.0 * (__builtin_fma(br, yi, -(bi * yr)) + __builtin_fma(cr, zi, -(ci * zr)));
    k[1] = k1;
    k[2] = k2;
    k[0] = -(k1 + k2);
    // C01 = h0 x + a p1 + b z^*,  C10 = a^* p0 + h1 x^* + c y^*
    const double c01r = __builtin_fma(h0, xr, __builtin_fma(ar, p1, __builtin_fma(br, zr, bi * zi)));
    const double c01i = __builtin_fma(h0, xi, __builtin_fma(ai, p1, __builtin_fma(bi, zr, -(br * zi))));
    const double c10r = __builtin_fma(ar, p0, __builtin_fma(h1, xr, __builtin_fma(cr, yr, ci * yi)));
    const double c10i = __builtin_fma(-ai, p0, __builtin_fma(-h1, xi, __builtin_fma(ci, yr, -(cr * yi))));
    k[3] = c01i + c10i;
    k[4] = c10r - c01r;
    // C02 = h0 y + a z + b p2,  C20 = b^* p0 + c^* x^* + h2 y^*
    const double c02r = __builtin_fma(h0, yr, __builtin_fma(ar, zr, __builtin_fma(-ai, zi, br * p2)));
    const double c02i = __builtin_fma(h0, yi, __builtin_fma(ar, zi, __builtin_fma(ai, zr, bi * p2)));
    const double c20r = __builtin_fma(br, p0, __builtin_fma(cr, xr, __builtin_fma(-ci, xi, h2 * yr)));
    const double c20i = __builtin_fma(-bi, p0, __builtin_fma(-cr, xi, __builtin_fma(-ci, xr, -(h2 * yi))));
    k[5] = c02i + c20i;
    k[6] = c20r - c02r;
    // C12 = a^* y + h1 z + c p2,  C21 = b^* x + c^* p1 + h2 z^*
    const double c12r = __builtin_fma(ar, yr, __builtin_fma(ai, yi, __builtin_fma(h1, zr, cr * p2)));
    const double c12i = __builtin_fma(ar, yi, __builtin_fma(-ai, yr, __builtin_fma(h1, zi, ci * p2)));
    const double c21r = __builtin_fma(br, xr, __builtin_fma(bi, xi, __builtin_fma(cr, p1, h2 * zr)));
    const double c21i = __builtin_fma(br, xi, __builtin_fma(-bi, xr, __builtin_fma(-ci, p1, -(h2 * zi))));
    k[7] = c12i + c21i;
    k[8] = c21r - c12r;
}

// Slopes of rho and rhobar (eq. eom): H = Hvac + Hmat + Hnn and
// Hbar = (Hvac - Hmat - Hnn)^*, hv and hvb holding Hvac + Hmat and
// Hvac - Hmat packed.
__device__ __forceinline__ void slope_of(const double hv[9], const double hvb[9], const double Hnn[9],
                                         const double y[18], double kk[18])
{
#pragma clang fp contract(off)
    double H[9], Hb[9];
#pragma unroll
    for (int k = 0; k < 9; k++) {
        H[k] = hv[k] + Hnn[k];
        const double hb = hvb[k] - Hnn[k];
        Hb[k] = (k == 4 || k == 6 || k == 8) ? -hb : hb;
    }
    commutator_fma(H, y, kk);
    commutator_fma(Hb, y + 9, kk + 9);
}

// Share of one direction's sources X (one particle per lane) that the lane's
// own cell takes with the weights of the anchor fraction ph; what leaves the
// tile goes to the direction's edge buffer ebd [edge][9].
template <int SH>
__device__ __forceinline__ void deposit_share(const double X[9], double ph, int lane, int nact, double xc[9],
                                              double *ebd)
{
    if (SH == 2) {
        // quadratic deposit: the particle at anchor m feeds cells m - 1 +
        // up' .. m + 1 + up', so cell m takes w0' w1' w2' of lanes (m + 1,
        // m, m - 1) when up' = 0 and of lanes (m, m - 1, m - 2) when up' = 1
        // (one-lane DPP moves); what leaves the tile goes to the edge
        // partials: one cell on the left (lane 0), two on the right (the
        // last active lanes)
        const Quad q = quad_weights(ph);
#pragma unroll
        for (int k = 0; k < 9; k++) {
            const double x = X[k];
            double s1 = lane_below(x);
            s1 = (lane == 0) ? 0.0 : s1;
            double a, b, c;
            if (q.up) {
                double s2 = lane_below(s1);
                s2 = (lane == 0) ? 0.0 : s2;
                a = x;
                b = s1;
                c = s2;
            } else {
                double xa = lane_above(x);
                xa = (lane == TILE - 1) ? 0.0 : xa;
                a = xa;
                b = x;
                c = s1;
            }
            xc[k] = wsum3(q.w0, a, q.w1, b, q.w2, c);
            if (lane == nact - 1) {
                ebd[0 * 9 + k] = q.up ? wsum2(q.w1, x, q.w2, s1) : q.w2 * x;
                ebd[1 * 9 + k] = q.up ? q.w2 * x : 0.0;
            }
            if (lane == 0)
                ebd[2 * 9 + k] = q.up ? 0.0 : q.w0 * x;
        }
    } else {
        // cell m gets (1 - phi') of its own particle and phi' of the
        // particle one lane to the left
        const double omph = 1.0 - ph;
#pragma unroll
        for (int k = 0; k < 9; k++) {
            double xl = lane_below(X[k]);
            xl = (lane == 0) ? 0.0 : xl;
            xc[k] = wsum2(omph, X[k], ph, xl);
        }
        if (lane == nact - 1) {
#pragma unroll
            for (int k = 0; k < 9; k++)
                ebd[k] = ph * X[k];
        }
    }
}

// The share as density and flux moments into the lane's 36 sums.
template <int SH>
__device__ __forceinline__ void deposit_dir(const double X[9], double ph, double vx, double vy, double vz,
                                            int lane, int nact, double acc[NG], double *ebd)
{
    double xc[9];
    deposit_share<SH>(X, ph, lane, nact, xc, ebd);
#pragma unroll
    for (int k = 0; k < 9; k++) {
        acc[k] += xc[k];
        acc[9 + k] += vx * xc[k];
        acc[18 + k] += vy * xc[k];
        acc[27 + k] += vz * xc[k];
    }
}

// LDS doubles of a workgroup's per-direction data (edge buffers, phi and
// (r, delta) tables), and of wg_reduce's buffer.
__host__ __device__ constexpr int dir_doubles(int nwaves, int max_dpw, int ne)
{
    return nwaves * max_dpw * (9 * ne + 3);
}
__host__ __device__ constexpr int red_doubles(int nwaves, int ne) { return NG * TILE + nwaves * NG * ne; }

// A workgroup's partials: the 36 sums of every lane over its waves, in wave
// order, to part, and each edge component over its directions (sgn: the sign
// of the flux groups), then over the waves, to edge.
template <int SH>
__device__ __forceinline__ void wg_reduce(const SimDesc &S, const WorkItem &wi, const double acc[NG],
                                          const double *eb, int dbeg, int dend, double sgn, double *red,
                                          int wave, int lane, int nwaves)
{
    constexpr int NE = n_edges(SH);
    __syncthreads();  // the grid tile is no longer needed: reuse it
    for (int w = 0; w < nwaves; ++w) {
        if (wave == w) {
#pragma unroll
            for (int k = 0; k < NG; k++)
                red[k * TILE + lane] = (w == 0) ? acc[k] : red[k * TILE + lane] + acc[k];
        }
        __syncthreads();
    }
    // edge partials of each wave: one lane per (edge, moment component) sums
    // over the wave's directions
    double *esum = red + NG * TILE;  // [nwaves][NE][NG]
    for (int q = lane; q < NE * NG; q += TILE) {
        const int e = q / NG, r = q - e * NG;
        const int comp = r % 9, grp = r / 9;
        double s = 0.0;
        for (int d = dbeg; d < dend; ++d) {
            // (values selected, not pointers: a select between fields of the
            // descriptor copy would put the whole copy in scratch memory)
            const double v1 = tld(S.vx, d), v2 = tld(S.vy, d), v3 = tld(S.vz, d);
            const double coef = (grp == 0) ? 1.0 : sgn * ((grp == 1) ? v1 : (grp == 2) ? v2 : v3);
            s += coef * eb[((d - dbeg) * NE + e) * 9 + comp];
        }
        esum[(wave * NE + e) * NG + r] = s;
    }
    __syncthreads();

    const int tile0 = wi.tile * TILE;
    const int ntc = S.ntile * TILE;
    double *part = S.part + (size_t)wi.group * NG * ntc;
    for (int idx = threadIdx.x; idx < NG * TILE; idx += blockDim.x) {
        const int k = idx / TILE, l = idx - k * TILE;
        gst(part + (size_t)k * ntc + tile0 + l, red[idx]);
    }
    for (int q = threadIdx.x; q < NE * NG; q += blockDim.x) {
        const int e = q / NG, r = q - e * NG;
        double s = 0.0;
        for (int w = 0; w < nwaves; ++w)
            s += esum[(w * NE + e) * NG + r];
        gst(S.edge + (((size_t)wi.group * NG + r) * NE + e) * S.ntile + wi.tile, s);
    }
}

// Sum over ng direction groups, stride apart, in group order (loads of eight
// groups in flight together).
__device__ __forceinline__ double group_sum(const double *p, int ng, size_t stride)
{
    double s = 0.0;
    int g = 0;
    for (; g + 8 <= ng; g += 8) {
        double v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q)
            v[q] = gld(p + (size_t)(g + q) * stride);
#pragma unroll
        for (int q = 0; q < 8; ++q)
            s += v[q];
    }
    for (; g < ng; ++g)
        s += gld(p + (size_t)g * stride);
    return s;
}

// Edge partials that reach cell l of a tile, as (source tile, edge slot)
// pairs in a fixed order; f(src, e) is called for each.  Linear: a tile's
// first cell takes the right edge of the tile before it (closing the periodic
// box).  Quadratic: a tile's right-edge cells are the first two after it (the
// second lies two tiles on when the next tile has one cell), its left-edge
// cell the last before it; with one tile or very few cells they fold onto the
// tile itself.  Candidate sources: tiles T-2, T-1, T, T+1 (each once); only a
// tile's first two cells and its last one take any.  (Periodic indices by
// compare and subtract: with integer divisions, tens of instructions each,
// the reduction of the 777 x 92 box took 13.9 us against 7 for the linear
// shape.)
template <class F>
__device__ __forceinline__ void edge_sources(int shape, int nc, int ntile, int tile, int l, F f)
{
    const int tm1 = tile == 0 ? ntile - 1 : tile - 1;
    if (shape != 2) {
        if (l == 0)
            f(tm1, 0);
        return;
    }
    const int tile0 = tile * TILE;
    if (l >= 2 && l != min(TILE, nc - tile0) - 1)
        return;
    const int j = tile0 + l;
    auto up = [](int x, int n) { return x >= n ? x - n : x; };
    const int tm2 = tm1 == 0 ? ntile - 1 : tm1 - 1;
    const int cand[4] = {tm2, tm1, tile, up(tile + 1, ntile)};
#pragma unroll
    for (int ci = 0; ci < 4; ++ci) {
        const int src = cand[ci];
        bool seen = false;
#pragma unroll
        for (int cj = 0; cj < ci; ++cj)
            seen = seen || (cand[cj] == src);
        if (seen)
            continue;
        const int t0s = src * TILE, nas = min(TILE, nc - t0s);
#pragma unroll 1
        for (int e = 0; e < 3; ++e) {
            const int target = (e < 2) ? up(up(t0s + nas + e, nc), nc) : up(t0s + nc - 1, nc);
            if (target == j)
                f(src, e);
        }
    }
}

}  // namespace fpic
