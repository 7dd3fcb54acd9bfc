// Wilson-fermion kernels: the hopping term H of M = 1 - kappa H and the fused
// even-odd CG on Mhat^dagger Mhat, Mhat = 1 - kappa^2 D_eo D_oe (FP64).
//
// The paper's second workload is an N_f = 2 Wilson-fermion program (Sec. 2, Sec. 6);
// it does not write the operator out, so the textbook form is used:
//   (H psi)(x) = sum_mu [(1 - gamma_mu) W_mu(x) psi(x + mu) + (1 + gamma_mu) W_mu(x - mu)^dagger psi(x - mu)],
//   W_mu(x) = s U_mu(x) (s: the t-boundary sign of the hop from x to x + mu),
// gamma matrices of a chiral basis with gamma_5 = diag(1, 1, -1, -1).
//
// Spin projection: 1 -+ gamma_mu has rank 2 in this basis, so each hop
// projects the neighbour's 4-spinor onto two spin components h0, h1, applies
// the 3x3 link to those only, and rebuilds spins 2 and 3 as multiples of
// them (half the colour arithmetic of the full product).
//
// Layout: links as for the staggered operator (the forward links of a site in
// tiles of 64 sites, FP64, two or three stored rows; the backward hop daggers
// the neighbour's); spinors of one parity as 12 planes of Vh complex
// (plane = 3 * spin + colour), a full field as [parity][12][Vh].  The template
// parameter LP reads the links: PrecF64 with plain loads, PrecF64NT with
// non-temporal ones for the backward neighbours' (fields whose links do not
// fit the Infinity Cache).
#pragma once

#include <type_traits>

#include "hop.hpp"

namespace stag {
namespace wil {

// ---- spin projection tables ---------------------------------------------------------
// Coefficients coded 0: 1, 1: -1, 2: i, 3: -i.
// Direction d = mu (forward, 1 - gamma_mu) or 4 + mu (backward, 1 + gamma_mu):
//   h0 = psi_0 + a0 psi_k0, h1 = psi_1 + a1 psi_k1;
//   result spins (h0, h1, b2 h_j2, b3 h_j3).
struct Proj {
    int k0, a0, k1, a1, j2, b2, j3, b3;
};
__device__ constexpr Proj kProj[8] = {
    {3, 3, 2, 3, 1, 2, 0, 2},  // mu = x, forward
    {3, 0, 2, 1, 1, 1, 0, 0},  // mu = y, forward
    {2, 3, 3, 2, 0, 2, 1, 3},  // mu = z, forward
    {2, 1, 3, 1, 0, 1, 1, 1},  // mu = t, forward
    {3, 2, 2, 2, 1, 3, 0, 3},  // mu = x, backward
    {3, 1, 2, 0, 1, 0, 0, 1},  // mu = y, backward
    {2, 2, 3, 3, 0, 3, 1, 2},  // mu = z, backward
    {2, 0, 3, 0, 0, 0, 1, 0},  // mu = t, backward
};

template <int C> __device__ __forceinline__ cplx<double> times(const cplx<double> &z)
{
    if constexpr (C == 0)
        return z;
    else if constexpr (C == 1)
        return {-z.re, -z.im};
    else if constexpr (C == 2)
        return {-z.im, z.re};
    else
        return {z.im, -z.re};
}

// z times the coefficient coded c, without branches (c may be a runtime value:
// the coefficient is formed by selects of constants, and the product by
// multiplications, so the gathers around it are not split into separate
// basic blocks that each wait for their loads)
__device__ __forceinline__ cplx<double> times(int c, const cplx<double> &z)
{
    const double cr = c == 0 ? 1.0 : (c == 1 ? -1.0 : 0.0);
    const double ci = c == 2 ? 1.0 : (c == 3 ? -1.0 : 0.0);
    return {z.re * cr - z.im * ci, z.re * ci + z.im * cr};
}

// The projector of direction d, 4 bits per field, so that a lane-dependent
// choice between directions is one select of a constant word.
__host__ __device__ constexpr uint32_t pack_proj(const Proj &q)
{
    return (uint32_t)q.k0 | (uint32_t)q.a0 << 4 | (uint32_t)q.k1 << 8 | (uint32_t)q.a1 << 12 | (uint32_t)q.j2 << 16 |
           (uint32_t)q.b2 << 20 | (uint32_t)q.j3 << 24 | (uint32_t)q.b3 << 28;
}

__device__ __forceinline__ Proj unpack_proj(uint32_t w)
{
    return {(int)(w & 15), (int)(w >> 4 & 15), (int)(w >> 8 & 15), (int)(w >> 12 & 15),
            (int)(w >> 16 & 15), (int)(w >> 20 & 15), (int)(w >> 24 & 15), (int)(w >> 28)};
}

// Projector of direction d.  The table is never read from memory: with d
// known at compile time (unrolled loop, one lane per site) the word is a
// constant, else it is chosen by selects among the candidates.
__device__ __forceinline__ Proj proj_of(int d)
{
    uint32_t w = pack_proj(kProj[0]);
#pragma unroll
    for (int t = 1; t < 8; ++t)
        w = d == t ? pack_proj(kProj[t]) : w;
    return unpack_proj(w);
}

// True when the t-boundary sign of Wilson hop d of the site with coordinates c
// is negative (the sign of the stored link it uses, forward or daggered).
__device__ __forceinline__ bool wilson_link_negative(const Geom &g, const SiteCoord &c, int d)
{
    const int ct = c.t, Lt = g.L[3], tap = g.tap;  // values first: the choice below is a select
    return tap && (d & 3) == 3 && (d >= 4 ? ct == 0 : ct == Lt - 1);
}

// acc[spin][colour] = (H psi)(s) for output site s of parity p_out, computed
// by LPS lanes (sub = 0 .. LPS-1; lane sub takes mu = sub, sub + LPS, ...,
// forward and backward; with LPS = 8 one hop each) and summed over them, so
// every lane of the site ends with the total.  lout / lin: the links of the
// output parity and of the other one.  load(n, sp, col) returns component
// (sp, col) of the input at site n of the other parity (with gamma_5 or any
// fused combination applied by the caller).
template <int ROWS, int LPS, class LP, class Load>
__device__ __forceinline__ void wilson_hop(const Geom &g, const dbl2 *__restrict__ lout, const dbl2 *__restrict__ lin,
                                           int p_out, int s, int sub, cplx<double> (&acc)[4][3], Load load)
{
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int a = 0; a < 3; ++a)
            acc[sp][a] = czero<double>();
    const SiteCoord c = decode_site(g, p_out, s);
    // one hop; kind 0: forward, 1: backward, 2: backward if d >= 4, by lane
    // (the matrix is then formed by selects, so lanes do not diverge)
    auto one_hop = [&](auto kind, int d) {
        constexpr int K = decltype(kind)::value;
        const bool back = K == 2 ? d >= 4 : K == 1;
        const int mu = d & 3;
        const Proj q = proj_of(d);
        const int n = neighbour(g, c, s, d);
        cplx<double> U[9];
        if constexpr (K == 1)
            load_link_rows<LP, ROWS, true>(lin + link_offset(ROWS, mu, n), U);
        else
            load_link_rows<LP, ROWS, false>((back ? lin : lout) + link_offset(ROWS, mu, back ? n : s), U);
        if constexpr (ROWS == 2)
            third_row(U, wilson_link_negative(g, c, d) ? -1.0 : 1.0);
        cplx<double> M[9];
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const cplx<double> u = U[a * 3 + b], v = U[b * 3 + a];
                M[a * 3 + b] = {back ? v.re : u.re, back ? -v.im : u.im};
            }
        cplx<double> h[2][3];
#pragma unroll
        for (int col = 0; col < 3; ++col) {
            const cplx<double> p0 = load(n, 0, col), p1 = load(n, 1, col);
            const cplx<double> pk0 = load(n, q.k0, col), pk1 = load(n, q.k1, col);  // spins 2, 3
            const cplx<double> t0 = times(q.a0, pk0), t1 = times(q.a1, pk1);
            h[0][col] = {p0.re + t0.re, p0.im + t0.im};
            h[1][col] = {p1.re + t1.re, p1.im + t1.im};
        }
        cplx<double> u[2][3];
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                u[k][a] = czero<double>();
#pragma unroll
                for (int b = 0; b < 3; ++b)
                    cmac(u[k][a], M[a * 3 + b], h[k][b]);
            }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            acc[0][a].re += u[0][a].re;
            acc[0][a].im += u[0][a].im;
            acc[1][a].re += u[1][a].re;
            acc[1][a].im += u[1][a].im;
            const cplx<double> r2 = times(q.b2, q.j2 ? u[1][a] : u[0][a]);
            const cplx<double> r3 = times(q.b3, q.j3 ? u[1][a] : u[0][a]);
            acc[2][a].re += r2.re;
            acc[2][a].im += r2.im;
            acc[3][a].re += r3.re;
            acc[3][a].im += r3.im;
        }
    };
    using fwd_t = std::integral_constant<int, 0>;
    using back_t = std::integral_constant<int, 1>;
    using lane_t = std::integral_constant<int, 2>;
    if constexpr (LPS == 1) {
        // two directions per iteration: enough loads in flight without spilling
#pragma unroll 1
        for (int mu = 0; mu < 4; ++mu) {
            one_hop(fwd_t{}, mu);
            one_hop(back_t{}, 4 + mu);
        }
    } else {
        if constexpr (LPS == 8) {
            one_hop(lane_t{}, sub);
        } else {
#pragma unroll
            for (int j = 0; j < 4 / LPS; ++j) {
                one_hop(fwd_t{}, sub + j * LPS);
                one_hop(back_t{}, 4 + sub + j * LPS);
            }
        }
#pragma unroll
        for (int sp = 0; sp < 4; ++sp)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                acc[sp][a].re = lane_sum<LPS>(acc[sp][a].re);
                acc[sp][a].im = lane_sum<LPS>(acc[sp][a].im);
            }
    }
}

// Component k = 3 * spin + colour of a site is handled by lane k mod LPS: lane
// sub has components sub, sub + LPS, ... (kOwn of them, the last one past the
// 12th for some lanes if LPS = 8).
template <int LPS> constexpr int kOwn = (12 + LPS - 1) / LPS;

// o[j] = component j LPS + sub of acc, by selects
template <int LPS>
__device__ __forceinline__ void own_components(const cplx<double> (&acc)[4][3], int sub, cplx<double> (&o)[kOwn<LPS>])
{
#pragma unroll
    for (int j = 0; j < kOwn<LPS>; ++j) {
        o[j] = acc[j * LPS / 3][j * LPS % 3];
#pragma unroll
        for (int t = 1; t < LPS; ++t) {
            const int k = j * LPS + t;
            if (k < 12) {
                const cplx<double> z = acc[k / 3][k % 3];
                o[j] = {sub == t ? z.re : o[j].re, sub == t ? z.im : o[j].im};
            }
        }
    }
}

// fn(j, k) for each component k of this lane, without branches between them
// (a branch per component made every load of an update wait for the one before)
template <int LPS, class Fn> __device__ __forceinline__ void each_own(int sub, Fn fn)
{
#pragma unroll
    for (int j = 0; j < kOwn<LPS>; ++j) {
        const int k = j * LPS + sub;
        if (12 % LPS == 0 || k < 12)
            fn(j, k);
    }
}

// Component k, or (spin, colour), of a 12-plane parity vector at site n.
__device__ __forceinline__ cplx<double> comp(const dbl2 *v, int Vh, int n, int k)
{
    const dbl2 t = v[(int64_t)k * Vh + n];
    return {t.x, t.y};
}

__device__ __forceinline__ cplx<double> comp(const dbl2 *v, int Vh, int n, int sp, int col)
{
    const dbl2 t = v[(int64_t)(sp * 3 + col) * Vh + n];
    return {t.x, t.y};
}

__device__ __forceinline__ void put(dbl2 *v, int Vh, int n, int k, const cplx<double> &z)
{
    v[(int64_t)k * Vh + n] = dbl2{z.re, z.im};
}

// Site and lane-within-site of this thread (LPS lanes per site, sub-major
// within a wavefront), false for threads past the last site.  With remap, the
// blocks of each XCD cover one contiguous range of sites (logical_block).
template <int LPS> __device__ __forceinline__ bool wsite(int Vh, int remap, int &s, int &sub)
{
    site_of_thread<LPS>((int)(logical_block(blockIdx.x, gridDim.x, remap) * blockDim.x + threadIdx.x), s, sub);
    return s < Vh;
}

// ---- the standalone hop: out_p = H_p in (one parity, or both, their blocks
// alternating so that the two uses of a link meet in one XCD's L2) ---------------------

template <int ROWS, int LPS, class LP>
__global__ void __launch_bounds__(128)
k_wilson_dslash(Geom g, const dbl2 *__restrict__ links, const dbl2 *__restrict__ in, dbl2 *__restrict__ out,
                int par_fixed, int remap)
{
    const BlockTile tl = block_tile(par_fixed >= 0 ? 1 : 2, remap, g.st * LPS / (int)blockDim.x);
    const int p = par_fixed >= 0 ? par_fixed : tl.tile;
    const int Vh = g.Vh;
    int s, sub;
    site_of_thread<LPS>(tl.chunk * blockDim.x + threadIdx.x, s, sub);
    if (s >= Vh)
        return;
    const dbl2 *src = in + (size_t)(1 - p) * 12 * Vh;
    cplx<double> acc[4][3];
    const int64_t lp = link_parity_entries(ROWS, Vh);
    wilson_hop<ROWS, LPS, LP>(g, links + lp * p, links + lp * (1 - p), p, s, sub, acc,
                          [&](int n, int sp, int col) { return comp(src, Vh, n, sp, col); });
    cplx<double> h[kOwn<LPS>];
    own_components<LPS>(acc, sub, h);
    dbl2 *o = out + (size_t)p * 12 * Vh;
    each_own<LPS>(sub, [&](int j, int k) { put(o, Vh, s, k, h[j]); });
}

// ---- even-odd CG ------------------------------------------------------------------

enum WMode : int32_t { W_IDLE = 0, W_INIT = 1, W_CG = 2, W_DONE = 3 };

struct WState {
    double stop2;  // tol^2 <rhs, rhs>
    double tol2;
    double bb;
    double rr;     // <r,r>
    double beta;
    double pad[3];
    int32_t mode;
    int32_t status;
    int32_t iters;
    int32_t maxiter;
    int32_t step;
    int32_t pad1[3];
};
static_assert(sizeof(WState) == 96, "state layout");

struct WArgs {
    Geom g;
    const dbl2 *links[2];  // per parity of their site
    double kappa;
    const dbl2 *b;         // caller's source [2][12][Vh]
    dbl2 *x;               // caller's solution [2][12][Vh]; even half iterated, odd half at the end
    dbl2 *bh;              // even: b_e + kappa D_eo b_o
    dbl2 *r;               // even
    dbl2 *p;               // even
    dbl2 *ap;              // even: Mhat p
    dbl2 *t;               // odd work vector
    WState *st[2];
    double *partials;      // [2 buffers][2 slots: 0 <ap,ap>, 1 <r,r>][pstride]
    int pstride;
    int remap;             // 1: XCD-contiguous site ranges (logical_block)
};

__device__ __forceinline__ double *wslot(const WArgs &a, int buf, int slot)
{
    return a.partials + ((size_t)buf * 2 + slot) * a.pstride;
}

// Totals of the first NS slots of partial buffer `buf` over nblk blocks,
// summed in a fixed order (strided per thread, then the wave and block trees).
template <int NS>
__device__ __forceinline__ void wtotals(const WArgs &a, int buf, int nblk, double *lds, double (&tot)[NS])
{
    double v[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k)
        v[k] = 0.0;
    for (int i0 = threadIdx.x; i0 < nblk; i0 += 4 * blockDim.x) {
        double q[4][NS];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * blockDim.x;
            const bool in = i < nblk;
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                const double v = wslot(a, buf, k)[in ? i : 0];  // in bounds; the guard selects
                q[u][k] = in ? v : 0.0;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k = 0; k < NS; ++k)
                v[k] += q[u][k];
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        const double t = wave_sum(v[k]);
        if (lane == 0)
            lds[k * nw + w] = t;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        double t = 0.0;
        for (int i = 0; i < nw; ++i)
            t += lds[k * nw + i];
        tot[k] = t;
    }
    __syncthreads();
}

// Block total of v into partial slot `slot` of buffer `buf` at this block.
__device__ __forceinline__ void wpartial(const WArgs &a, int buf, int slot, double v, double *lds)
{
    double arr[1] = {v};
    double out;
    block_sum_multi<1>(arr, lds, out);
    if (threadIdx.x == 0)
        wslot(a, buf, slot)[blockIdx.x] = out;
}

__device__ __forceinline__ bool wfinite_pos(double v) { return v > 0.0 && v < INFINITY; }

__device__ __forceinline__ int wuniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ double wuniform(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// init 1 (even outputs): bh = b_e + kappa (H b)_e
template <int ROWS, int LPS, class LP> __global__ void __launch_bounds__(128) k_wil_bhat(WArgs a)
{
    const int Vh = a.g.Vh;
    int s, sub;
    if (!wsite<LPS>(Vh, a.remap, s, sub))
        return;
    const dbl2 *bo = a.b + (size_t)12 * Vh;
    cplx<double> acc[4][3];
    wilson_hop<ROWS, LPS, LP>(a.g, a.links[0], a.links[1], 0, s, sub, acc,
                          [&](int n, int sp, int col) { return comp(bo, Vh, n, sp, col); });
    cplx<double> h[kOwn<LPS>];
    own_components<LPS>(acc, sub, h);
    each_own<LPS>(sub, [&](int j, int k) {
        const cplx<double> be = comp(a.b, Vh, s, k);
        put(a.bh, Vh, s, k, {be.re + a.kappa * h[j].re, be.im + a.kappa * h[j].im});
    });
}

// odd outputs: t = H_oe (gamma_5 src).  With a state (K3 of a step) it runs
// only while the system iterates; without one (initialisation) always.
template <int ROWS, int LPS, class LP>
__global__ void __launch_bounds__(128) k_wil_odd_g5(WArgs a, const dbl2 *__restrict__ src, int ver, int check)
{
    if (check && a.st[ver ^ 1]->mode != W_CG)
        return;
    const int Vh = a.g.Vh;
    int s, sub;
    if (!wsite<LPS>(Vh, a.remap, s, sub))
        return;
    cplx<double> acc[4][3];
    wilson_hop<ROWS, LPS, LP>(a.g, a.links[1], a.links[0], 1, s, sub, acc, [&](int n, int sp, int col) {
        const cplx<double> z = comp(src, Vh, n, sp, col);
        return sp < 2 ? z : cplx<double>{-z.re, -z.im};
    });
    cplx<double> h[kOwn<LPS>];
    own_components<LPS>(acc, sub, h);
    each_own<LPS>(sub, [&](int j, int k) { put(a.t, Vh, s, k, h[j]); });
}

// init 3 (even outputs): r = bh - kappa^2 gamma_5 (H t)_e = Mhat^dagger bh;
// x_e = 0; <r,r> into slot 1 of buffer 0
template <int ROWS, int LPS, class LP> __global__ void __launch_bounds__(128) k_wil_init(WArgs a)
{
    __shared__ double lds[4];
    const int Vh = a.g.Vh;
    int s, sub;
    double nrm = 0.0;
    if (wsite<LPS>(Vh, a.remap, s, sub)) {
        cplx<double> acc[4][3];
        wilson_hop<ROWS, LPS, LP>(a.g, a.links[0], a.links[1], 0, s, sub, acc,
                              [&](int n, int sp, int col) { return comp(a.t, Vh, n, sp, col); });
        cplx<double> h[kOwn<LPS>];
        own_components<LPS>(acc, sub, h);
        const double k2 = a.kappa * a.kappa;
        each_own<LPS>(sub, [&](int j, int k) {
            const double g5 = k < 6 ? k2 : -k2;
            const cplx<double> bh = comp(a.bh, Vh, s, k);
            const cplx<double> r = {bh.re - g5 * h[j].re, bh.im - g5 * h[j].im};
            put(a.r, Vh, s, k, r);
            put(a.x, Vh, s, k, czero<double>());
            nrm += r.re * r.re + r.im * r.im;
        });
    }
    wpartial(a, 0, 1, nrm, lds);
}

// A step, with ap = Mhat p carried by a recurrence (ap' = Mhat r + beta ap for
// p' = r + beta p; its relative rounding is that of the recurrence of p):
//   K1  t = H_oe r, no scalar needed;
//   K2  beta, then ap' = r - kappa^2 H_eo t + beta ap and <ap',ap'>;
//   K3  t = H_oe gamma_5 ap';
//   K4  alpha, then p' = r + beta p, x += alpha p', r -= alpha Mhat^dagger ap'
//       (= ap' - kappa^2 gamma_5 H_eo t) and <r,r>.
// The direct form gathered r and p at every neighbour in K1 (3 KB a site
// instead of 1.5), and its prologue ran before K1's hop.  K2 and K4 sum the
// partials after their hop: at 16^4 a block needs 10 us for a hop from the
// Infinity Cache and L2, and with the totals before it and a branch per
// component of the update K2 took 19.2 us and K4 20.9, now 12.2 and 14.5.

// K1 (odd outputs): t = H_oe r while the system iterates (or has not begun)
template <int ROWS, int LPS, class LP> __global__ void __launch_bounds__(128) k_wil_step1(WArgs a, int ver)
{
    const int mode = a.st[ver]->mode;
    if (mode != W_CG && mode != W_INIT)
        return;
    const int Vh = a.g.Vh;
    int s, sub;
    if (!wsite<LPS>(Vh, a.remap, s, sub))
        return;
    cplx<double> acc[4][3];
    wilson_hop<ROWS, LPS, LP>(a.g, a.links[1], a.links[0], 1, s, sub, acc,
                              [&](int n, int sp, int col) { return comp(a.r, Vh, n, sp, col); });
    cplx<double> h[kOwn<LPS>];
    own_components<LPS>(acc, sub, h);
    each_own<LPS>(sub, [&](int j, int k) { put(a.t, Vh, s, k, h[j]); });
}

// K2 (even outputs): advance the state over the previous step, then
// ap' = r - kappa^2 (H t)_e + beta ap; <ap',ap'> into slot 0 of buffer ver^1
template <int ROWS, int LPS, class LP> __global__ void __launch_bounds__(128) k_wil_step2(WArgs a, int ver)
{
    __shared__ double lds[8];
    __shared__ __align__(16) WState sst;
    const int Vh = a.g.Vh, nblk = gridDim.x;
    const int mode0 = a.st[ver]->mode;
    if (mode0 != W_CG && mode0 != W_INIT) {
        if (blockIdx.x == 0 && threadIdx.x == 0)
            *a.st[ver ^ 1] = *a.st[ver];  // pass the final state on
        return;
    }
    if (threadIdx.x < sizeof(WState) / 16)
        ((uint4 *)&sst)[threadIdx.x] = ((const uint4 *)a.st[ver])[threadIdx.x];
    // the hop and the site's own vectors need no scalar: they come before the
    // totals, so that the waits for the two overlap
    int s, sub;
    const bool site = wsite<LPS>(Vh, a.remap, s, sub);
    cplx<double> h[kOwn<LPS>], o[kOwn<LPS>];
    if (site) {
        cplx<double> acc[4][3];
        wilson_hop<ROWS, LPS, LP>(a.g, a.links[0], a.links[1], 0, s, sub, acc,
                                  [&](int n, int sp, int col) { return comp(a.t, Vh, n, sp, col); });
        own_components<LPS>(acc, sub, h);
        const double k2 = a.kappa * a.kappa;
        each_own<LPS>(sub, [&](int j, int k) {
            const cplx<double> r = comp(a.r, Vh, s, k);
            o[j] = comp(a.ap, Vh, s, k);
            h[j] = {r.re - k2 * h[j].re, r.im - k2 * h[j].im};
        });
    }
    double tot[2];
    wtotals<2>(a, ver, nblk, lds, tot);  // its barriers also publish sst
    if (threadIdx.x == 0) {
        WState st = sst;
        st.step += 1;
        if (st.mode == W_INIT) {
            const double bb = tot[1];
            st.bb = bb;
            st.rr = bb;
            st.stop2 = st.tol2 * bb;
            st.beta = 0.0;
            st.iters = 0;
            if (!(bb < INFINITY)) {
                st.mode = W_DONE;
                st.status = STAG_ENONFINITE;
            } else if (bb == 0.0) {
                st.mode = W_DONE;
                st.status = STAG_OK;
            } else if (st.maxiter == 0) {
                st.mode = W_DONE;
                st.status = STAG_ENOCONV;
            } else {
                st.mode = W_CG;
            }
        } else {
            const double pap = tot[0], rn = tot[1];
            st.iters += 1;
            if (!wfinite_pos(pap) || !(rn < INFINITY)) {
                st.mode = W_DONE;
                st.status = STAG_EBREAKDOWN;
            } else if (rn < st.stop2) {
                st.rr = rn;
                st.mode = W_DONE;
                st.status = STAG_OK;
            } else if (st.iters >= st.maxiter) {
                st.rr = rn;
                st.mode = W_DONE;
                st.status = STAG_ENOCONV;
            } else {
                st.beta = rn / st.rr;
                st.rr = rn;
            }
        }
        if (blockIdx.x == 0)
            *a.st[ver ^ 1] = st;
        sst = st;
    }
    __syncthreads();
    if (wuniform(sst.mode) != W_CG)
        return;
    const double beta = wuniform(sst.beta);
    double nrm = 0.0;
    if (site) {
        each_own<LPS>(sub, [&](int j, int k) {
            if (beta != 0.0)  // beta = 0 starts from ap = 0, whatever the buffer holds
                h[j] = {fma(beta, o[j].re, h[j].re), fma(beta, o[j].im, h[j].im)};
            put(a.ap, Vh, s, k, h[j]);
            nrm += h[j].re * h[j].re + h[j].im * h[j].im;
        });
    }
    wpartial(a, ver ^ 1, 0, nrm, lds);
}

// K4 (even outputs): alpha = rr / <ap',ap'>; p' = r + beta p; atap = ap' -
// kappa^2 gamma_5 (H t)_e (= Mhat^dagger Mhat p'); x += alpha p'; r -= alpha
// atap; <r,r> into slot 1 of buffer ver^1
template <int ROWS, int LPS, class LP> __global__ void __launch_bounds__(128) k_wil_step4(WArgs a, int ver)
{
    __shared__ double lds[8];
    const WState *st = a.st[ver ^ 1];
    if (st->mode != W_CG)
        return;
    const int cur = ver ^ 1;
    const double rr = wuniform(st->rr), beta = wuniform(st->beta);
    const int Vh = a.g.Vh;
    int s, sub;
    const bool site = wsite<LPS>(Vh, a.remap, s, sub);
    cplx<double> h[kOwn<LPS>], r[kOwn<LPS>], p[kOwn<LPS>], x[kOwn<LPS>];
    if (site) {  // before the totals, as in K2
        cplx<double> acc[4][3];
        wilson_hop<ROWS, LPS, LP>(a.g, a.links[0], a.links[1], 0, s, sub, acc,
                                  [&](int n, int sp, int col) { return comp(a.t, Vh, n, sp, col); });
        own_components<LPS>(acc, sub, h);
        const double k2 = a.kappa * a.kappa;
        each_own<LPS>(sub, [&](int j, int k) {
            const double g5 = k < 6 ? k2 : -k2;
            const cplx<double> ap = comp(a.ap, Vh, s, k), o = comp(a.p, Vh, s, k);
            r[j] = comp(a.r, Vh, s, k);
            x[j] = comp(a.x, Vh, s, k);
            h[j] = {ap.re - g5 * h[j].re, ap.im - g5 * h[j].im};
            p[j] = r[j];
            if (beta != 0.0)  // beta = 0 starts from p = 0
                p[j] = {fma(beta, o.re, r[j].re), fma(beta, o.im, r[j].im)};
        });
    }
    double tot[1];
    wtotals<1>(a, cur, gridDim.x, lds, tot);
    const double alpha = wfinite_pos(tot[0]) ? rr / tot[0] : 0.0;
    double nrm = 0.0;
    if (site) {
        each_own<LPS>(sub, [&](int j, int k) {
            put(a.p, Vh, s, k, p[j]);
            put(a.x, Vh, s, k, {fma(alpha, p[j].re, x[j].re), fma(alpha, p[j].im, x[j].im)});
            const cplx<double> rn = {fma(-alpha, h[j].re, r[j].re), fma(-alpha, h[j].im, r[j].im)};
            put(a.r, Vh, s, k, rn);
            nrm += rn.re * rn.re + rn.im * rn.im;
        });
    }
    wpartial(a, cur, 1, nrm, lds);
}

// x_o = b_o + kappa (H x_e)_o
template <int ROWS, int LPS, class LP> __global__ void __launch_bounds__(128) k_wil_xodd(WArgs a)
{
    const int Vh = a.g.Vh;
    int s, sub;
    if (!wsite<LPS>(Vh, a.remap, s, sub))
        return;
    cplx<double> acc[4][3];
    wilson_hop<ROWS, LPS, LP>(a.g, a.links[1], a.links[0], 1, s, sub, acc,
                          [&](int n, int sp, int col) { return comp(a.x, Vh, n, sp, col); });
    const dbl2 *bo = a.b + (size_t)12 * Vh;
    dbl2 *xo = a.x + (size_t)12 * Vh;
    cplx<double> h[kOwn<LPS>];
    own_components<LPS>(acc, sub, h);
    each_own<LPS>(sub, [&](int j, int k) {
        const cplx<double> b = comp(bo, Vh, s, k);
        put(xo, Vh, s, k, {b.re + a.kappa * h[j].re, b.im + a.kappa * h[j].im});
    });
}

// |b - M x|^2 on the sites of parity `par`, per block into slot `par` of
// buffer 0 (the solve is over when this runs)
template <int ROWS, int LPS, class LP> __global__ void __launch_bounds__(128) k_wil_resid(WArgs a, int par)
{
    __shared__ double lds[4];
    const int Vh = a.g.Vh;
    int s, sub;
    double nrm = 0.0;
    if (wsite<LPS>(Vh, a.remap, s, sub)) {
        const dbl2 *xin = a.x + (size_t)(1 - par) * 12 * Vh;
        cplx<double> acc[4][3];
        wilson_hop<ROWS, LPS, LP>(a.g, a.links[par], a.links[1 - par], par, s, sub, acc,
                              [&](int n, int sp, int col) { return comp(xin, Vh, n, sp, col); });
        const dbl2 *bp = a.b + (size_t)par * 12 * Vh;
        const dbl2 *xp = a.x + (size_t)par * 12 * Vh;
        cplx<double> h[kOwn<LPS>];
        own_components<LPS>(acc, sub, h);
        each_own<LPS>(sub, [&](int j, int k) {
            const cplx<double> b = comp(bp, Vh, s, k), x = comp(xp, Vh, s, k);
            const double re = b.re - x.re + a.kappa * h[j].re;
            const double im = b.im - x.im + a.kappa * h[j].im;
            nrm += re * re + im * im;
        });
    }
    wpartial(a, 0, par, nrm, lds);
}

}  // namespace wil
}  // namespace stag
