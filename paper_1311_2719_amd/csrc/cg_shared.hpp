// CG step kernels for FP32 and FP16 working precision in which the systems
// of a tile share every link read through LDS.
//
// The register tiles of cg_kernels.hpp share a link load between the R
// systems one thread carries, so their per-thread state grows with R and the
// tuner settles on R = 2 or 3 at 24^4: every link is then read from HBM
// S / R times per kernel.  Here a block is W wavefronts, each running RR
// systems of the block's tile (R = W RR) on 64 consecutive output sites, one
// lane per site.  The block first reads the links of those 64 sites (8
// directions, stored rows), rebuilds row 2 where only two are stored,
// converts them to FP32 and keeps all nine entries in LDS; every wavefront
// then runs the hop of its RR systems with the links taken from there.  A
// link thus costs one HBM read per R systems (R up to 16: one tile per parity
// at 12 or 16 systems), the third row and the FP16 conversion are computed
// once per block instead of once per thread, and a wavefront holds the
// registers of RR systems only.
//
// The step arithmetic is that of k_cg_step1 / k_cg_step2 (the loop of the
// paper's Sec. 4 with the mass explicit; FP32 the recurrence of u = D p, FP16
// the direct form): same products, same storage
// formats, same state machine (advance()); only the summation order of the
// partial sums differs (each system's sums stay in one wavefront: lane sums
// over the chunks a block visits, then the wavefront sum).
//
// LDS layout of one chunk: [entry 9][dir 8][site 64 + 8] of FP32 complex.  A
// wavefront reading one (entry, dir) for its 64 sites touches 512 contiguous
// bytes; the 8 padding entries per row put the eight directions of one
// staging store in different banks.
#pragma once

#include "cg_kernels.hpp"

namespace stag {

constexpr int kChunk = 64;              // output sites per block and round
constexpr int kLdsRow = kChunk + 8;     // padded row of one (entry, dir)
constexpr int kSharedMaxR = 16;         // systems per tile
// Directions of the hop whose gathers a wavefront keeps in flight together,
// and the wavefronts per SIMD the register allocation must allow.  A fully
// unrolled hop holds the gathers of all eight directions (about 130 VGPRs);
// occupancy, not unrolling, hides the gather latency here.  The residual
// recomputation (FP64, rare) runs its direction loop rolled so that it does
// not set the kernel's register budget.
constexpr int kSharedDirUnroll = 2;
constexpr int kSharedMinWaves = 1;

__device__ __forceinline__ int chunk_link_index(int k, int d, int i) { return (k * 8 + d) * kLdsRow + i; }

// Staging of the matrices of the 8 hops of output sites [s0, s0 + 64) (parity
// p_out) into lk: W_mu(s) for the forward hops, -W_mu(s - mu)^dagger for the
// backward ones.  A wavefront takes one hop of the 64 sites, so its loads and
// its LDS stores are contiguous (the backward neighbours of 64 consecutive
// sites are consecutive but for the x direction's and the boundaries' steps).
// Two parts, so that the step's prologue runs while the first loads are in
// flight: load() starts the loads of a wavefront's first kPre hops, store()
// writes them to LDS and does the rest.  A smaller tile runs at the tuned
// shape's block count, which may exceed the chunks: a block without a chunk
// (chunk_start() = -1) loads the first sites' links, never stores them, and
// writes partial sums of zero.
template <class P, int ROWS, int W> struct ChunkLinks {
    static constexpr int kPre = (8 + W - 1) / W <= 2 ? (8 + W - 1) / W : 1;
    SiteCoord c;
    int s;
    cplx<float> U[kPre][9];

    static __device__ __forceinline__ int wave() { return uniform((int)(threadIdx.x >> 6)); }

    __device__ __forceinline__ void load_hop(const Geom &g, const typename P::link_t *lout,
                                             const typename P::link_t *lin, int d, cplx<float> (&u)[9])
    {
        const bool back = d >= 4;
        load_link_rows<P, ROWS, false>(
            (back ? lin : lout) + link_offset(ROWS, d & 3, back ? neighbour(g, c, s, d) : s), u);
    }
    __device__ __forceinline__ void load(const Geom &g, const typename P::link_t *lout, const typename P::link_t *lin,
                                         int p_out, int s0)
    {
        s = (s0 < 0 ? 0 : s0) + (threadIdx.x & 63);
        s = s < g.Vh ? s : g.Vh - 1;  // past the end: staged, never used
        c = decode_site(g, p_out, s);
#pragma unroll
        for (int k = 0; k < kPre; ++k)
            if (wave() + k * W < 8)
                load_hop(g, lout, lin, wave() + k * W, U[k]);
    }
    __device__ __forceinline__ void store_hop(const Geom &g, int d, cplx<float> (&u)[9], flt2 *lk)
    {
        const bool back = d >= 4;
        if constexpr (ROWS == 2)
            third_row(u, folded_negative(g, c, d) != back ? -2.f : 2.f);
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const cplx<float> f = u[a * 3 + b], t = u[b * 3 + a];
                lk[chunk_link_index(a * 3 + b, d, threadIdx.x & 63)] = back ? flt2{-t.re, t.im} : flt2{f.re, f.im};
            }
    }
    __device__ __forceinline__ void store(const Geom &g, const typename P::link_t *lout, const typename P::link_t *lin,
                                          flt2 *lk)
    {
#pragma unroll
        for (int k = 0; k < kPre; ++k)
            if (wave() + k * W < 8)
                store_hop(g, wave() + k * W, U[k], lk);
        for (int d = wave() + kPre * W; d < 8; d += W) {
            cplx<float> u[9];
            load_hop(g, lout, lin, d, u);
            store_hop(g, d, u, lk);
        }
    }
};

// acc[q][a] += sum_d L_d(s)[a][b] chi_qd[b] for the RR systems of a
// wavefront, the links from the staged chunk (lane i = site s0 + i),
// load(q, n, chi) the input of system q at neighbour n.
template <bool TABLES, int RR, class Load>
__device__ __forceinline__ void hop_shared_impl(const Geom &g, const int32_t *__restrict__ nbr, int p_out, int s,
                                                int i, const flt2 *lk, cplx<float> (&acc)[RR][3], Load load)
{
    SiteCoord c;
    if constexpr (!TABLES)
        c = decode_site(g, p_out, s);
#pragma unroll kSharedDirUnroll
    for (int d = 0; d < 8; ++d) {
        int n;
        if constexpr (TABLES)
            n = nbr[(int64_t)d * g.Vh + s];
        else
            n = neighbour(g, c, s, d);
        cplx<float> chi[RR][3];
#pragma unroll
        for (int q = 0; q < RR; ++q)
            load(q, n, chi[q]);
        cplx<float> U[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const flt2 v = lk[chunk_link_index(k, d, i)];
            U[k] = {v.x, v.y};
        }
#pragma unroll
        for (int q = 0; q < RR; ++q)
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int b = 0; b < 3; ++b)
                    cmac(acc[q][a], U[a * 3 + b], chi[q][b]);
    }
}

template <int RR, class Load>
__device__ __forceinline__ void hop_shared(const Geom &g, const int32_t *nbr, int p_out, int s, int i, const flt2 *lk,
                                           cplx<float> (&acc)[RR][3], Load load)
{
    if (nbr)
        hop_shared_impl<true, RR>(g, nbr, p_out, s, i, lk, acc, load);
    else
        hop_shared_impl<false, RR>(g, nbr, p_out, s, i, lk, acc, load);
}

// Totals of slots [0, NS) of system j's partial sums (the previous kernel's
// per-block sums), formed by one wavefront:
// lane l adds entries l, l + 64, ... in order, then the wavefront sum.
template <int NS> __device__ __forceinline__ void wave_prologue_sums(const CgArgs &a, int buf, int j, double (&t)[NS])
{
    const int lane = threadIdx.x & 63;
    double v[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k)
        v[k] = 0.0;
    for (int i = lane; i < a.nread; i += 64)
#pragma unroll
        for (int k = 0; k < NS; ++k)
            v[k] += partial_slot(a, buf, j, k)[i];
#pragma unroll
    for (int k = 0; k < NS; ++k)
        t[k] = wave_sum(v[k]);
}

// First site of the chunk a block takes in round `it`, or -1 past the end.
__device__ __forceinline__ int chunk_start(int it, int Vh, const StepTile &tl)
{
    const int64_t s0 = ((int64_t)it * tl.nchunks + tl.chunk) * kChunk;
    return s0 < Vh ? (int)s0 : -1;
}

// ---- K1 -----------------------------------------------------------------------------
// A block of W wavefronts runs a tile of R = W RR systems; wavefront w takes
// places w RR .. w RR + RR - 1.  Like the register tiles, a wavefront gathers
// for each of its places, also places whose system is not in a CG step (their
// sums are discarded), so that the direction loop has no per-system branch.

template <class P, int W, int RR, int ROWS>
__global__ void __launch_bounds__(64 * W, kSharedMinWaves) k_cg_shared1(CgArgs a, int ver)
{
    constexpr int R = W * RR;
    static_assert(P::id != 0 && R <= kSharedMaxR, "shared-link tiles: FP32 / FP16 working precision");
    using real = typename P::real;
    using v2 = typename vec2_of<real>::type;
    __shared__ flt2 lk[9 * 8 * kLdsRow];
    __shared__ int modes[R];
    const StepTile tl = step_tile<R>(a, a.g.st, kChunk);
    const int par = tl.par, k0 = tl.k0, pout = 1 - par;
    const int Vh = a.g.Vh;
    // the wavefront index is the same in every lane: kept in a scalar register,
    // so that its systems, their states and pointers stay scalar too
    const int w = uniform((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    bool anyplace = false;
#pragma unroll
    for (int r = 0; r < R; ++r)
        anyplace |= a.perm[k0 + r] >= 0;
    if (!anyplace)
        return;
    const auto *lout = (const typename P::link_t *)a.links[pout], *lin = (const typename P::link_t *)a.links[1 - pout];
    ChunkLinks<P, ROWS, W> cl;
    cl.load(a.g, lout, lin, pout, chunk_start(0, Vh, tl));
    // prologue: this wavefront advances its own systems over the previous step
    int js[RR];
    bool cg[RR], ru[RR];
    real beta[RR];
    int pc[RR];
#pragma unroll
    for (int q = 0; q < RR; ++q) {
        const int j = a.perm[k0 + w * RR + q];
        int mode = M_IDLE, p = 0;
        double b = 0.0;
        if (j >= 0 && a.nread == 0) {  // k_cg_scalars has advanced the state
            const SysState &st = a.st[ver ^ 1][j];
            mode = st.mode;
            b = st.beta;
            p = st.pcur;
        } else if (j >= 0) {
            double t[3];
            wave_prologue_sums<3>(a, ver, j, t);
            SysState st = a.st[ver][j];
            const bool live = st.mode != M_IDLE && st.mode != M_DONE;
            if (live)
                advance<kRecurrence<P>>(st, t);
            // the state K2 of this step reads: advanced, or the same idle/done state
            if (tl.chunk == 0 && lane == 0)
                a.st[ver ^ 1][j] = st;
            mode = live ? uniform(st.mode) : (int)M_IDLE;
            b = uniform(st.beta);
            p = uniform(st.pcur);
        }
        js[q] = j;
        cg[q] = mode == M_CG;
        ru[q] = mode == M_RU;
        beta[q] = (real)b;
        pc[q] = p;
        if (lane == 0)
            modes[w * RR + q] = mode;
    }
    __syncthreads();
    bool anycg = false, anyru = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        anycg |= modes[r] == M_CG;
        anyru |= modes[r] == M_RU;
    }
    if (!anycg && !anyru)
        return;
    bool wcg = false;
#pragma unroll
    for (int q = 0; q < RR; ++q)
        wcg |= cg[q];
    // every place gathers in bounds: an empty place reads system 0's vectors
    const v2 *rv[RR];
    const void *pold[RR];
    void *uv[RR];
#pragma unroll
    for (int q = 0; q < RR; ++q) {
        const int jj = js[q] >= 0 ? js[q] : 0;
        rv[q] = (const v2 *)a.r + (size_t)jj * 3 * Vh;
        pold[q] = spin_at<P>(a.p[kRecurrence<P> ? 0 : pc[q]], jj, Vh);
        uv[q] = spin_at<P>(a.ap, jj, Vh);
    }
    double nrm_ap[RR], nrm_p[RR];
#pragma unroll
    for (int q = 0; q < RR; ++q)
        nrm_ap[q] = nrm_p[q] = 0.0;
    for (int it = 0;; ++it) {
        const int s0 = chunk_start(it, Vh, tl);
        if (s0 < 0)
            break;
        if (anycg) {
            if (it > 0) {
                __syncthreads();  // every wavefront is done with the previous chunk's links
                cl.load(a.g, lout, lin, pout, s0);
            }
            cl.store(a.g, lout, lin, lk);
            __syncthreads();
        }
        const int s = s0 + lane;
        if (s >= Vh)
            continue;
        if (wcg) {
            cplx<float> acc[RR][3];
#pragma unroll
            for (int q = 0; q < RR; ++q)
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    acc[q][c] = czero<float>();
            if constexpr (kRecurrence<P>) {
                // u at this site: before the gathers for a single system, after them for several
                cplx<real> uo[RR][3];
                auto own = [&]() {
#pragma unroll
                    for (int q = 0; q < RR; ++q)
                        P::load_spinor(uv[q], Vh, s, uo[q]);
                };
                if constexpr (RR == 1)
                    own();
                auto load = [&](int q, int n, cplx<float> *chi) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const v2 t = rv[q][(int64_t)c * Vh + n];
                        chi[c] = {t.x, t.y};
                    }
                };
                hop_shared<RR>(a.g, a.nbr[pout], pout, s, lane, lk, acc, load);
                if constexpr (RR > 1)
                    own();
#pragma unroll
                for (int q = 0; q < RR; ++q) {
                    if (!cg[q])
                        continue;
                    cplx<real> un[3];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        // beta = 0 starts from u = 0, whatever the buffer holds
                        un[c].re = beta[q] != 0.f ? fmaf(beta[q], uo[q][c].re, acc[q][c].re) : acc[q][c].re;
                        un[c].im = beta[q] != 0.f ? fmaf(beta[q], uo[q][c].im, acc[q][c].im) : acc[q][c].im;
                        nrm_ap[q] += (double)un[c].re * un[c].re + (double)un[c].im * un[c].im;
                    }
                    P::store_spinor(uv[q], Vh, s, un);
                }
            } else {
                // the partner site's p and r (same index, parity par): before the
                // gathers for a single system, after them for several
                cplx<real> po[RR][3];
                v2 ro[RR][3];
                auto own = [&]() {
#pragma unroll
                    for (int q = 0; q < RR; ++q) {
                        P::load_spinor(pold[q], Vh, s, po[q]);
#pragma unroll
                        for (int c = 0; c < 3; ++c)
                            ro[q][c] = rv[q][(int64_t)c * Vh + s];
                    }
                };
                if constexpr (RR == 1)
                    own();
                auto load = [&](int q, int n, cplx<float> *chi) {
                    cplx<real> pv[3];
                    P::load_spinor(pold[q], Vh, n, pv);
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const v2 t = rv[q][(int64_t)c * Vh + n];
                        chi[c].re = fma(beta[q], pv[c].re, t.x);
                        chi[c].im = fma(beta[q], pv[c].im, t.y);
                    }
                };
                hop_shared<RR>(a.g, a.nbr[pout], pout, s, lane, lk, acc, load);
                if constexpr (RR > 1)
                    own();
#pragma unroll
                for (int q = 0; q < RR; ++q) {
                    if (!cg[q])
                        continue;
                    const int j = js[q];
                    cplx<real> pn[3];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        pn[c].re = fma(beta[q], po[q][c].re, ro[q][c].x);
                        pn[c].im = fma(beta[q], po[q][c].im, ro[q][c].y);
                    }
                    P::store_spinor(spin_at<P>(a.ap, j, Vh), Vh, s, acc[q]);
                    void *pnew = spin_at<P>(a.p[pc[q] ^ 1], j, Vh);
                    P::store_spinor_read_back(pnew, Vh, s, pn);  // pn: the value D will read
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        nrm_p[q] += (double)pn[c].re * pn[c].re + (double)pn[c].im * pn[c].im;
                        nrm_ap[q] += (double)acc[q][c].re * acc[q][c].re + (double)acc[q][c].im * acc[q][c].im;
                    }
                }
            }
        }
    }
    // residual recomputations (FP64, rare) after the CG work, by the whole
    // block: eight lanes per site, one direction each
    for (int r = 0; anyru && r < R; ++r) {
        if (modes[r] != M_RU)
            continue;
        const int j = a.perm[k0 + r];
        for (int it = 0;; ++it) {
            const int s0 = chunk_start(it, Vh, tl);
            if (s0 < 0)
                break;
            for (int t = threadIdx.x; t < kChunk * 8; t += blockDim.x) {  // whole wavefronts
                int sl, sub;
                site_of_thread<8>(t, sl, sub);
                if (s0 + sl < Vh)
                    recompute_k1<8, ROWS>(a, j, pout, s0 + sl, sub);
            }
        }
    }
    if (!anycg)
        return;
#pragma unroll
    for (int q = 0; q < RR; ++q) {
        if (js[q] < 0)
            continue;
        const double tap = wave_sum(nrm_ap[q]);
        if (lane == 0)
            partial_slot(a, ver ^ 1, js[q], 0)[tl.chunk] = tap;
        if constexpr (!kRecurrence<P>) {
            const double tpp2 = wave_sum(nrm_p[q]);
            if (lane == 0)
                partial_slot(a, ver ^ 1, js[q], 1)[tl.chunk] = tpp2;
        }
    }
}

// ---- K2 -----------------------------------------------------------------------------

template <class P, int W, int RR, int ROWS>
__global__ void __launch_bounds__(64 * W, kSharedMinWaves) k_cg_shared2(CgArgs a, int ver)
{
    constexpr int R = W * RR;
    static_assert(P::id != 0 && R <= kSharedMaxR, "shared-link tiles: FP32 / FP16 working precision");
    using real = typename P::real;
    using v2 = typename vec2_of<real>::type;
    __shared__ flt2 lk[9 * 8 * kLdsRow];
    __shared__ int modes[R];
    __shared__ double red[2 * W];
    const StepTile tl = step_tile<R>(a, a.g.st, kChunk);
    const int par = tl.par, k0 = tl.k0;
    const int Vh = a.g.Vh;
    const int cur = ver ^ 1;  // the state K1 of this step wrote
    // the wavefront index is the same in every lane: kept in a scalar register,
    // so that its systems, their states and pointers stay scalar too
    const int w = uniform((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    bool anyplace = false;
#pragma unroll
    for (int r = 0; r < R; ++r)
        anyplace |= a.perm[k0 + r] >= 0;
    if (!anyplace)
        return;
    const auto *lout = (const typename P::link_t *)a.links[par], *lin = (const typename P::link_t *)a.links[1 - par];
    ChunkLinks<P, ROWS, W> cl;
    cl.load(a.g, lout, lin, par, chunk_start(0, Vh, tl));
    // alpha from K1's partial sums (slot 0; FP16: slots 0 and 1)
    constexpr int NS = kRecurrence<P> ? 1 : 2;
    int js[RR], pn_buf[RR];
    bool cg[RR], ru[RR];
    real al[RR], be[RR], m2r[RR];
    double m2[RR];
#pragma unroll
    for (int q = 0; q < RR; ++q) {
        const int j = a.perm[k0 + w * RR + q];
        int mode = M_IDLE, pb = 0;
        double alpha = 0.0, beta = 0.0, mass2 = 0.0;
        if (j >= 0) {
            const SysState &st = a.st[cur][j];
            const int smode = st.mode;
            const double rr = st.rr;
            const int pcur = st.pcur;
            mass2 = st.mass2;
            beta = uniform(st.beta);
            const double pp = st.pp;
            double t[NS];
            if (a.nread != 0)
                wave_prologue_sums<NS>(a, cur, j, t);
            if (smode == M_CG && a.nread == 0) {
                alpha = st.alpha;  // 0: <p',Ap'> was not a positive number
                mode = alpha != 0.0 ? (int)M_CG : (int)M_IDLE;
            } else if (smode == M_CG) {
                const double pap = mass2 * (kRecurrence<P> ? pp : t[NS - 1]) + t[0];
                if (finite_pos(pap)) {  // otherwise K1 of the next step reports the breakdown
                    mode = M_CG;
                    alpha = rr / pap;
                }
            } else if (smode == M_RU) {
                mode = M_RU;
            }
            mode = uniform(mode);
            alpha = uniform(alpha);
            mass2 = uniform(mass2);
            pb = kRecurrence<P> ? 0 : uniform(pcur) ^ 1;  // FP16: p' written by K1 of this step
        }
        js[q] = j;
        cg[q] = mode == M_CG;
        ru[q] = mode == M_RU;
        al[q] = (real)alpha;
        be[q] = (real)beta;
        m2[q] = mass2;
        m2r[q] = (real)mass2;
        pn_buf[q] = pb;
        if (lane == 0)
            modes[w * RR + q] = mode;
    }
    __syncthreads();
    bool anycg = false, anyru = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        anycg |= modes[r] == M_CG;
        anyru |= modes[r] == M_RU;
    }
    if (!anycg && !anyru)
        return;
    bool wcg = false;
#pragma unroll
    for (int q = 0; q < RR; ++q)
        wcg |= cg[q];
    const void *apv[RR];
#pragma unroll
    for (int q = 0; q < RR; ++q)
        apv[q] = spin_at<P>(a.ap, js[q] >= 0 ? js[q] : 0, Vh);
    double nrm[RR], nrp[RR];  // <r,r>; <r,p'> (recurrence form)
#pragma unroll
    for (int q = 0; q < RR; ++q)
        nrm[q] = nrp[q] = 0.0;
    for (int it = 0;; ++it) {
        const int s0 = chunk_start(it, Vh, tl);
        if (s0 < 0)
            break;
        if (anycg) {
            if (it > 0) {
                __syncthreads();
                cl.load(a.g, lout, lin, par, s0);
            }
            cl.store(a.g, lout, lin, lk);
            __syncthreads();
        }
        const int s = s0 + lane;
        if (s >= Vh)
            continue;
        if (wcg) {
            // this site's p (FP16: p'), x and r: before the gathers for a single system,
            // after them for several
            cplx<real> pv[RR][3];
            flt2 xv[RR][3];
            v2 ro[RR][3];
            auto own_as = [&](auto nt) {
                constexpr bool NT = decltype(nt)::value;
#pragma unroll
                for (int q = 0; q < RR; ++q) {
                    if (!cg[q])
                        continue;
                    const int j = js[q];
                    const void *pb = spin_at<P>(a.p[pn_buf[q]], j, Vh);
                    if constexpr (!kRecurrence<P>)
                        P::load_spinor(pb, Vh, s, pv[q]);
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        if constexpr (kRecurrence<P>) {
                            const v2 t = load_own<NT>((const v2 *)pb + (int64_t)c * Vh + s);
                            pv[q][c] = {t.x, t.y};
                        }
                        xv[q][c] = load_own<NT>(&a.xlo[(size_t)j * 3 * Vh + (int64_t)c * Vh + s]);
                        ro[q][c] = ((const v2 *)a.r)[(size_t)j * 3 * Vh + (int64_t)c * Vh + s];
                    }
                }
            };
            auto own = [&]() { by_access(a.nt_vectors, own_as); };
            if constexpr (RR == 1)
                own();
            cplx<float> acc[RR][3];
#pragma unroll
            for (int q = 0; q < RR; ++q)
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    acc[q][c] = czero<float>();
            auto load = [&](int q, int n, cplx<float> *chi) { P::load_spinor(apv[q], Vh, n, chi); };
            hop_shared<RR>(a.g, a.nbr[par], par, s, lane, lk, acc, load);
            if constexpr (RR > 1)
                own();
#pragma unroll
            for (int q = 0; q < RR; ++q) {
                if (!cg[q])
                    continue;
                const int j = js[q];
                v2 *rv = (v2 *)a.r + (size_t)j * 3 * Vh;
                flt2 *xl = a.xlo + (size_t)j * 3 * Vh;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const int64_t o = (int64_t)c * Vh + s;
                    if constexpr (kRecurrence<P>) {
                        // p' = r + beta p; beta = 0 starts from p = 0, whatever the buffer holds
                        pv[q][c].re = be[q] != 0.f ? fmaf(be[q], pv[q][c].re, ro[q][c].x) : ro[q][c].x;
                        pv[q][c].im = be[q] != 0.f ? fmaf(be[q], pv[q][c].im, ro[q][c].y) : ro[q][c].y;
                    }
                    xv[q][c] = flt2{fmaf(al[q], pv[q][c].re, xv[q][c].x), fmaf(al[q], pv[q][c].im, xv[q][c].y)};
                    const real apr = m2r[q] * pv[q][c].re - acc[q][c].re;
                    const real api = m2r[q] * pv[q][c].im - acc[q][c].im;
                    v2 rn = ro[q][c];
                    rn.x = fma(-al[q], apr, rn.x);
                    rn.y = fma(-al[q], api, rn.y);
                    rv[o] = rn;
                    nrm[q] += (double)rn.x * rn.x + (double)rn.y * rn.y;
                    if constexpr (kRecurrence<P>)
                        nrp[q] += (double)rn.x * pv[q][c].re + (double)rn.y * pv[q][c].im;
                }
                by_access(a.nt_vectors, [&](auto nt) {
                    constexpr bool NT = decltype(nt)::value;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const int64_t o = (int64_t)c * Vh + s;
                        store_own<NT>(xv[q][c], &xl[o]);
                        if constexpr (kRecurrence<P>)
                            store_own<NT>(v2{pv[q][c].re, pv[q][c].im}, (v2 *)spin_at<P>(a.p[0], j, Vh) + o);
                    }
                });
            }
        }
    }
    // residual recomputations (FP64, rare) after the CG work, by the whole
    // block (see K1); each one's partial sum is the block's total
    for (int r = 0; anyru && r < R; ++r) {
        if (modes[r] != M_RU)
            continue;
        const int j = a.perm[k0 + r];
        const double m2d = a.st[cur][j].mass2;
        double nr[2] = {0.0, 0.0};
        for (int it = 0;; ++it) {
            const int s0 = chunk_start(it, Vh, tl);
            if (s0 < 0)
                break;
            for (int t = threadIdx.x; t < kChunk * 8; t += blockDim.x) {  // whole wavefronts
                int sl, sub;
                site_of_thread<8>(t, sl, sub);
                if (s0 + sl < Vh)
                    recompute_k2<P, 8, ROWS>(a, j, par, s0 + sl, sub, m2d, nr[0], nr[1]);
            }
        }
        double tot;
        block_sum_multi<2>(nr, red, tot);
        if (threadIdx.x == 0)
            partial_slot(a, cur, j, 2)[tl.chunk] = tot;
        if (kRecurrence<P> && threadIdx.x == 1)
            partial_slot(a, cur, j, 1)[tl.chunk] = tot;
    }
#pragma unroll
    for (int q = 0; q < RR; ++q) {
        if (js[q] < 0 || ru[q])
            continue;
        const double tot = wave_sum(nrm[q]);
        if (lane == 0)
            partial_slot(a, cur, js[q], 2)[tl.chunk] = tot;
        if constexpr (kRecurrence<P>) {
            const double trp = wave_sum(nrp[q]);
            if (lane == 0)
                partial_slot(a, cur, js[q], 1)[tl.chunk] = trp;
        }
    }
}

}  // namespace stag
