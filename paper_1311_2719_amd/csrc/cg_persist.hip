// The whole CG loop of one right-hand side in one launch, for lattices whose
// links fit the register files (the loop of the paper's Sec. 4; the same
// recurrence form, state machine and FP64 residual recomputations as the step
// kernels of cg_kernels.hpp).
//
// On small lattices a step kernel is bound by what surrounds its hop: the
// launch, the first loads of states and sums, the last block.  Here each lane
// keeps the links of its hops and its site's r, p, x and u in registers for the
// whole solve.  A step then moves r and u only, and its two grid-wide sums are
// also its two barriers.
//
// One lane group (LPS lanes) per site of the whole lattice: a site of parity
// q forms u of the system on parity 1 - q (K1) and updates p, x, r of the
// system on parity q (K2).  What sites exchange (r and u; in a residual
// recomputation x and D x) travels through memory: agent-scope (sc1) stores
// write through the XCD's L2 and agent-scope loads bypass it, so no cache has
// to be written back or invalidated.
//
// The sum of a value over all blocks: each block publishes its partial as two
// words {32 data bits, sequence number}, so that a reader that sees the
// sequence number has the data; the partial is published after the block's
// stores of r or u have completed, so the sum is a barrier for them too.  Up to
// kFlatBlocks blocks, every block reads all partials; beyond, one block per
// group of kGroup sums its group's partials and every block reads the group
// sums (256 blocks reading 256 partials of 4 values each took 14 us; 64 take
// 4).  All blocks add the same numbers in the same order.
//
// Every wait is bounded: a block that waits longer than kWaitTicks raises the
// abort word and leaves, the others follow, and the host repeats the solve with
// the step kernels.  The grids that the host lets run at a time on a device (of
// this process) have at most one block per CU together, so their blocks become
// resident once other kernels' blocks have ended.
//
// A step takes 7 us on one block (4^4), 9 at 8^4, 13 at 12^3 16 and 18 at 16^4
// in FP64: two chains of a gather, a block sum, a store that has to complete
// and a poll that sees it, about a microsecond each.  Solves, step kernels ->
// one launch: FP64 8^4 1.38 -> 0.84 ms, 6 10 14 8 1.44 -> 0.90, 12^3 16 2.29 -> 1.69,
// 16^4 3.31 -> 2.44; FP32 1.30 -> 0.87, 1.41 -> 0.91, 2.24 -> 1.52, 2.64 -> 1.71.
#include <algorithm>
#include <cstdlib>

#include "batch.hpp"
#include "cg_kernels.hpp"
#include "cg_persist.hpp"

namespace stag {

namespace {

constexpr int kThreads = 512;            // per block: two wavefronts per SIMD, 256 registers each
constexpr int kFlatBlocks = 64;          // blocks that read each other's partials directly
constexpr int kGroup = 32;               // blocks per group beyond that
constexpr int kCopies = 8;               // copies of the group sums, each read by 1/8 of the blocks
constexpr int kMaxBlocks = 256;
constexpr int kMaxGroups = kMaxBlocks / kGroup;
constexpr uint64_t kWaitTicks = 30000000;  // of the 100 MHz counter: 0.3 s
constexpr int kAgent = 16;               // cache policy of a buffer access: sc1

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

struct PersistArgs {
    CgArgs c;
    unsigned long long *slots;  // [2][4 values][kMaxBlocks][2], then [2][kCopies][4][kMaxGroups][2]
    int *abort;
    uint32_t seq0;              // sequence numbers seq0 + 1, ... have not been used
    int max_steps;
    uint64_t wait_ticks;        // longest wait for another block
};

constexpr int kBlockWords = 2 * 4 * kMaxBlocks * 2;
constexpr int kGroupWords = 2 * kCopies * 4 * kMaxGroups * 2;

__device__ __forceinline__ void publish(unsigned long long *p, double v, uint32_t seq)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v), tag = (uint64_t)seq << 32;
    __hip_atomic_store(p, (b & 0xffffffffu) | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(p + 1, (b >> 32) | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wait for the value published at p under `seq`; false when the wait is over
// without it.
__device__ __forceinline__ bool receive(const unsigned long long *p, uint32_t seq, uint64_t t0, const PersistArgs &pa,
                                        double &v)
{
    for (int spin = 0;; ++spin) {
        const uint64_t lo = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t hi = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((uint32_t)(lo >> 32) == seq && (uint32_t)(hi >> 32) == seq) {
            v = __builtin_bit_cast(double, (lo & 0xffffffffu) | (hi << 32));
            return true;
        }
        if ((spin & 63) == 63 && (wall_clock64() - t0 >= pa.wait_ticks ||
                                  __hip_atomic_load(pa.abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0))
            return false;
    }
}

// Agent-scope access to a vector of one parity: [colour 3][Vh] complex.
template <class P> struct Shared {
    using real = typename P::real;
    __amdgpu_buffer_rsrc_t rsrc;
    int Vh;
    __device__ __forceinline__ Shared(void *base, int vh) : Vh(vh)
    {
        rsrc = __builtin_amdgcn_make_buffer_rsrc(base, 0, 3 * vh * (int)(2 * sizeof(real)), 0x00027000);
    }
    __device__ __forceinline__ cplx<real> load(int s, int c) const
    {
        const int o = (c * Vh + s) * (int)(2 * sizeof(real));
        if constexpr (P::id == 0) {
            const dbl2 v = __builtin_bit_cast(dbl2, __builtin_amdgcn_raw_buffer_load_b128(rsrc, o, 0, kAgent));
            return {v.x, v.y};
        } else {
            const flt2 v = __builtin_bit_cast(flt2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, o, 0, kAgent));
            return {v.x, v.y};
        }
    }
    __device__ __forceinline__ void store(int s, int c, const cplx<real> &z) const
    {
        const int o = (c * Vh + s) * (int)(2 * sizeof(real));
        if constexpr (P::id == 0)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, dbl2{z.re, z.im}), rsrc, o, 0, kAgent);
        else
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, flt2{z.re, z.im}), rsrc, o, 0, kAgent);
    }
};

// The two grid-wide sums of a step and their scratch.  A wavefront has terms
// of one system only: even wavefronts of system `first`, odd ones of the other.
struct GridSum {
    const PersistArgs &pa;
    double *lds;   // [2][kThreads / 64]
    double *tot;   // [4]
    int *dead;
    uint32_t seq;

    // tot[j * N + n] = the sum over the grid of v[n] of system j; also a barrier
    // for the earlier agent-scope stores.  False: the wait was given up and the
    // block must leave.
    template <int N> __device__ __forceinline__ bool sum(const double (&v)[N], int first)
    {
        constexpr int NV = 2 * N;
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = kThreads / 64;
        const int nblk = (int)gridDim.x, b = (int)blockIdx.x;
        ++seq;
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const double t = wave_sum(v[n]);
            if (lane == 0)
                lds[n * nw + w] = t;
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wavefront's stores have completed
        __syncthreads();
        unsigned long long *mine = pa.slots + (size_t)(seq & 1) * (4 * kMaxBlocks * 2);
        if (threadIdx.x < NV) {
            const int j = threadIdx.x / N, n = threadIdx.x % N;
            double t = 0.0;
#pragma unroll
            for (int i = 0; i < nw; i += 2)
                t += lds[n * nw + i + (j ^ first)];
            publish(mine + ((size_t)threadIdx.x * kMaxBlocks + b) * 2, t, seq);
        }
        if (w < NV) {  // wavefront k receives value k
            const uint64_t t0 = wall_clock64();
            double s = 0.0, q;
            bool ok = pa.wait_ticks != 0;  // 0: given up before the first look
            if (nblk <= kFlatBlocks) {
                if (ok && lane < nblk) {
                    ok = receive(mine + ((size_t)w * kMaxBlocks + lane) * 2, seq, t0, pa, q);
                    s = ok ? q : 0.0;
                }
            } else {
                const int ng = (nblk + kGroup - 1) / kGroup;
                unsigned long long *grp = pa.slots + kBlockWords + (size_t)(seq & 1) * (kCopies * 4 * kMaxGroups * 2);
                if (b % kGroup == 0) {
                    double g = 0.0;
                    if (ok && lane < kGroup && b + lane < nblk) {
                        ok = receive(mine + ((size_t)w * kMaxBlocks + b + lane) * 2, seq, t0, pa, q);
                        g = ok ? q : 0.0;
                    }
                    g = wave_sum(g);
                    if (__all(ok) && lane < kCopies)
                        publish(grp + (((size_t)lane * 4 + w) * kMaxGroups + b / kGroup) * 2, g, seq);
                }
                if (ok && lane < ng) {
                    ok = receive(grp + (((size_t)(b % kCopies) * 4 + w) * kMaxGroups + lane) * 2, seq, t0, pa, q);
                    s = ok ? q : 0.0;
                }
            }
            if (!__all(ok)) {
                if (lane == 0) {
                    *dead = 1;
                    __hip_atomic_store(pa.abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            s = wave_sum(s);
            if (lane == 0)
                tot[w] = s;
        }
        __syncthreads();
        return *dead == 0;
    }
};

template <class P, int LPS, int ROWS>
__global__ void __launch_bounds__(kThreads, 2) k_cg_persist(PersistArgs pa)
{
    using real = typename P::real;
    using v2 = typename vec2_of<real>::type;
    static_assert(LPS == 2 || LPS == 4, "hops of a lane: mu = sub, sub + LPS, forward and backward");
    constexpr int HOPS = 8 / LPS, NO = LPS == 2 ? 2 : 1;  // colours a lane owns: sub, sub + LPS
    __shared__ double lds[2 * kThreads / 64];
    __shared__ double tot[4], uu[2];
    __shared__ __align__(16) SysState st[2];
    __shared__ int dead;
    const CgArgs &a = pa.c;
    const Geom &g = a.g;
    const int Vh = g.Vh, lane = threadIdx.x & 63;
    const int W = uniform((int)(blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6)));
    const int par = W & 1, oth = 1 - par;  // parity of this lane's site = its K2 system; its K1 system
    const int sub = lane / (64 / LPS), s0 = (W >> 1) * (64 / LPS) + lane % (64 / LPS);
    const bool in = s0 < Vh;
    const int s = in ? s0 : 0;
    if (threadIdx.x == 0)
        dead = 0;
    if (threadIdx.x < 2)
        st[threadIdx.x] = a.st[0][threadIdx.x];
    GridSum gs{pa, lds, tot, &dead, pa.seq0};
    // the links of this lane's hops, for the whole solve
    const SiteCoord c = decode_site(g, par, s);
    typename P::link_t U[HOPS][3 * ROWS];
    int nb[HOPS];
    real inv_c[HOPS];
    {
        const auto *lout = (const typename P::link_t *)a.links[par], *lin = (const typename P::link_t *)a.links[oth];
#pragma unroll
        for (int h = 0; h < HOPS; ++h) {
            const int mu = sub + (h >> 1) * LPS;
            const bool back = h & 1;
            nb[h] = neighbour(g, c, s, back ? mu + 4 : mu);
            inv_c[h] = folded_negative(g, c, back ? mu + 4 : mu) != back ? real(-2) : real(2);
            const auto *lp = (back ? lin : lout) + link_offset(ROWS, mu, back ? nb[h] : s);
#pragma unroll
            for (int k = 0; k < 3 * ROWS; ++k)
                U[h][k] = lp[k * kLinkTile];
        }
    }
    auto hop = [&](const Shared<P> &v, cplx<real> (&acc)[3]) {
        // the loads of PRE hops in flight: all but with four FP64 hops, whose
        // registers would spill
        constexpr int PRE = P::id == 0 && HOPS == 4 ? 2 : HOPS;
        cplx<real> chi[HOPS][3];
#pragma unroll
        for (int q = 0; q < 3; ++q)
            acc[q] = czero<real>();
#pragma unroll
        for (int h = 0; h < HOPS; ++h) {
            if (h % PRE == 0) {
                if (h > 0)
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = h; i < h + PRE; ++i)
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        chi[i][q] = v.load(nb[i], q);
            }
            cplx<real> M[9];
#pragma unroll
            for (int k = 0; k < 3 * ROWS; ++k)
                M[k] = {U[h][k].x, U[h][k].y};
            if constexpr (ROWS == 2)
                third_row(M, inv_c[h]);
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    if (h & 1)
                        cmsub_conj(acc[k], M[i * 3 + k], chi[h][i]);
                    else
                        cmac(acc[i], M[i * 3 + k], chi[h][k]);
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            acc[q].re = lane_sum<LPS>(acc[q].re);
            acc[q].im = lane_sum<LPS>(acc[q].im);
        }
    };
    // D of an FP64 vector (residual recomputations): with the links of the
    // solve in FP64, else with the FP64 links, one hop's loads at a time
    auto hop64 = [&](const Shared<PrecF64> &v, cplx<double> (&acc)[3]) {
        if constexpr (P::id == 0) {
            hop(v, acc);
        } else {
#pragma unroll
            for (int q = 0; q < 3; ++q)
                acc[q] = czero<double>();
#pragma unroll
            for (int h = 0; h < HOPS; ++h) {
                const int mu = sub + (h >> 1) * LPS;
                cplx<double> M[9], chi[3];
                load_link_rows<PrecF64, ROWS, false>(a.links64[h & 1 ? oth : par] + link_offset(ROWS, mu, h & 1 ? nb[h] : s),
                                                     M);
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    chi[q] = v.load(nb[h], q);
                if constexpr (ROWS == 2)
                    third_row(M, (double)inv_c[h]);
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int k = 0; k < 3; ++k)
                        if (h & 1)
                            cmsub_conj(acc[k], M[i * 3 + k], chi[i]);
                        else
                            cmac(acc[i], M[i * 3 + k], chi[k]);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                acc[q].re = lane_sum<LPS>(acc[q].re);
                acc[q].im = lane_sum<LPS>(acc[q].im);
            }
        }
    };
    // this lane's colours of a sum every lane holds
    auto owned = [&](const auto &acc, int q) {
        const int col = sub + q * LPS;
        auto z = acc[2];
        z.re = col == 0 ? acc[0].re : col == 1 ? acc[1].re : z.re;
        z.im = col == 0 ? acc[0].im : col == 1 ? acc[1].im : z.im;
        return z;
    };
    auto owns = [&](int q) { return in && sub + q * LPS < 3; };
    auto off = [&](int q) { return (int64_t)(sub + q * LPS) * Vh + s; };
    v2 *rm = (v2 *)a.r + (size_t)par * 3 * Vh;
    v2 *pm = (v2 *)spin_at<P>(a.p[0], par, Vh);
    v2 *um = (v2 *)spin_at<P>(a.ap, oth, Vh);
    // x in memory: the solution itself, or the mixed solve's low part
    v2 *xm = nullptr;
    if constexpr (P::id == 0)
        xm = (v2 *)a.xhi[par];
    else
        xm = (v2 *)(a.xlo + (size_t)par * 3 * Vh);
    const Shared<P> r_own((void *)rm, Vh), r_oth((v2 *)a.r + (size_t)oth * 3 * Vh, Vh);
    const Shared<P> u_oth((void *)um, Vh), u_own(spin_at<P>(a.ap, par, Vh), Vh);
    const Shared<PrecF64> x_own((void *)a.xhi[par], Vh), x_oth((void *)a.xhi[oth], Vh);
    const Shared<PrecF64> t_own(a.tmp + (size_t)par * 3 * Vh, Vh), t_oth(a.tmp + (size_t)oth * 3 * Vh, Vh);
    __syncthreads();
    cplx<real> r[NO], p[NO], x[NO], u[NO];
    double own_rr = 0.0, own_rp = 0.0;  // this lane's terms for its K2 system
    const bool init = st[par].mode == M_INIT;
    const bool solved = st[par].mode != M_IDLE;
#pragma unroll
    for (int q = 0; q < NO; ++q) {
        r[q] = p[q] = x[q] = u[q] = czero<real>();
        if (!owns(q))
            continue;
        if (solved && init) {
            const dbl2 bv = a.b[par][off(q)];
            x_own.store(s, sub + q * LPS, czero<double>());
            r[q] = p[q] = {(real)bv.x, (real)bv.y};
            own_rr += bv.x * bv.x + bv.y * bv.y;
        } else if (solved) {
            const v2 rv = rm[off(q)], pv = pm[off(q)], xv = xm[off(q)];
            r[q] = {rv.x, rv.y};
            p[q] = {pv.x, pv.y};
            x[q] = {xv.x, xv.y};
        }
        if (st[oth].mode == M_CG || st[oth].mode == M_RU) {
            const v2 uv = um[off(q)];
            u[q] = {uv.x, uv.y};
        }
        if (solved)
            r_own.store(s, sub + q * LPS, r[q]);
    }
    // the first sum: <b,b> of new systems, and every site's r is in place
    if (!gs.sum<2>({own_rr, own_rp}, 0))
        return;
    if (threadIdx.x < 2 && st[threadIdx.x].mode == M_INIT) {
        const double t[3] = {0.0, 0.0, tot[threadIdx.x * 2]};
        advance<true>(st[threadIdx.x], t);
    }
    __syncthreads();
    for (int step = 0; step < pa.max_steps; ++step) {
        const int m_own = uniform(st[par].mode), m_oth = uniform(st[oth].mode);
        const bool ru = m_own == M_RU || m_oth == M_RU;
        if (m_own != M_CG && m_oth != M_CG && !ru)
            break;
        if (ru) {  // a recomputation gathers x; the mixed solve's low part joins it first
            if (m_own == M_RU) {
#pragma unroll
                for (int q = 0; q < NO; ++q) {
                    if (!owns(q))
                        continue;
                    cplx<double> xn = {(double)x[q].re, (double)x[q].im};
                    if constexpr (P::id != 0) {
                        const cplx<double> hi = x_own.load(s, sub + q * LPS);
                        xn = {hi.re + xn.re, hi.im + xn.im};
                        x[q] = czero<real>();
                    }
                    x_own.store(s, sub + q * LPS, xn);
                }
            }
            if (!gs.sum<1>({0.0}, 0))
                return;
        }
        // K1: u of the other parity's system at this site
        double oth_uu = 0.0;
        if (m_oth == M_CG) {
            const real beta = (real)st[oth].beta;
            cplx<real> acc[3];
            hop(r_oth, acc);
#pragma unroll
            for (int q = 0; q < NO; ++q) {
                if (!owns(q))
                    continue;
                const cplx<real> d = owned(acc, q);
                u[q] = beta != real(0) ? cplx<real>{fma(beta, u[q].re, d.re), fma(beta, u[q].im, d.im)} : d;
                u_oth.store(s, sub + q * LPS, u[q]);
                oth_uu += (double)u[q].re * u[q].re + (double)u[q].im * u[q].im;
            }
        } else if (m_oth == M_RU) {  // t = D x
            cplx<double> acc[3];
            hop64(x_oth, acc);
#pragma unroll
            for (int q = 0; q < NO; ++q)
                if (owns(q))
                    t_oth.store(s, sub + q * LPS, owned(acc, q));
        }
        if (!gs.sum<1>({oth_uu}, 1))
            return;
        if (threadIdx.x < 2)
            uu[threadIdx.x] = tot[threadIdx.x];
        // K2: p, x and r of this parity's system
        own_rr = own_rp = 0.0;
        const double m2d = st[par].mass2;
        if (m_own == M_CG) {
            const double pap = m2d * st[par].pp + tot[par];
            if (finite_pos(pap)) {  // otherwise advance() reports the breakdown
                const real alpha = (real)(st[par].rr / pap), beta = (real)st[par].beta, m2 = (real)m2d;
                cplx<real> acc[3];
                hop(u_own, acc);
#pragma unroll
                for (int q = 0; q < NO; ++q) {
                    if (!owns(q))
                        continue;
                    const cplx<real> d = owned(acc, q);
                    p[q] = beta != real(0) ? cplx<real>{fma(beta, p[q].re, r[q].re), fma(beta, p[q].im, r[q].im)} : r[q];
                    x[q] = {fma(alpha, p[q].re, x[q].re), fma(alpha, p[q].im, x[q].im)};
                    r[q] = {fma(-alpha, m2 * p[q].re - d.re, r[q].re), fma(-alpha, m2 * p[q].im - d.im, r[q].im)};
                    r_own.store(s, sub + q * LPS, r[q]);
                    own_rr += (double)r[q].re * r[q].re + (double)r[q].im * r[q].im;
                    own_rp += (double)r[q].re * p[q].re + (double)r[q].im * p[q].im;
                }
            }
        } else if (m_own == M_RU) {  // r = b - m^2 x + D t
            cplx<double> acc[3];
            hop64(t_own, acc);
#pragma unroll
            for (int q = 0; q < NO; ++q) {
                if (!owns(q))
                    continue;
                const cplx<double> d = owned(acc, q), xv = x_own.load(s, sub + q * LPS);
                const dbl2 bv = a.b[par][off(q)];
                const double re = bv.x - m2d * xv.re + d.re, im = bv.y - m2d * xv.im + d.im;
                r[q] = {(real)re, (real)im};
                r_own.store(s, sub + q * LPS, r[q]);
                own_rr += re * re + im * im;
                own_rp += re * p[q].re + im * p[q].im;
            }
        }
        if (!gs.sum<2>({own_rr, own_rp}, 0))
            return;
        if (threadIdx.x < 2) {
            const int j = threadIdx.x;
            if (st[j].mode != M_IDLE && st[j].mode != M_DONE) {
                const double t[3] = {uu[j], tot[j * 2 + 1], tot[j * 2]};
                advance<true>(st[j], t);
            }
        }
        __syncthreads();
    }
    // what a further launch starts from
    const bool more = st[par].mode == M_CG || st[par].mode == M_RU;
#pragma unroll
    for (int q = 0; q < NO; ++q) {
        if (!owns(q))
            continue;
        if (more) {
            rm[off(q)] = v2{r[q].re, r[q].im};
            pm[off(q)] = v2{p[q].re, p[q].im};
            xm[off(q)] = v2{x[q].re, x[q].im};
        }
        um[off(q)] = v2{u[q].re, u[q].im};
    }
    if (blockIdx.x == 0 && threadIdx.x < 2) {
        a.st[0][threadIdx.x] = st[threadIdx.x];
        a.st[1][threadIdx.x] = st[threadIdx.x];
    }
}

template <class P, int LPS, int ROWS> hipError_t launch(const PersistArgs &pa, int nblk, hipStream_t s)
{
    hipLaunchKernelGGL((k_cg_persist<P, LPS, ROWS>), dim3((unsigned)nblk), dim3(kThreads), 0, s, pa);
    return hipGetLastError();
}

int blocks_for_lps(const Geom &g, int lps)
{
    const int64_t waves = 2 * (((int64_t)g.Vh * lps + 63) / 64);
    return (int)((waves * 64 + kThreads - 1) / kThreads);
}

}  // namespace

LaunchGate &persist_gate(int device)
{
    static LaunchGate gate[64];
    return gate[device & 63];
}

size_t cg_persist_bytes() { return (size_t)(kBlockWords + kGroupWords) * 8 + 256; }

// Two lanes per site hold four hops' links each, four lanes two: beyond
// 65536 sites the registers of 256 blocks do not hold the lattice, and three
// FP64 rows do not fit with two lanes.  Four lanes where all blocks still read
// each other's partials (FP64 solve, four / two lanes: 6 10 14 8 0.90 / 0.96 ms,
// 12^3 16, 216 / 108 blocks, 2.19 / 1.69; FP32 within 2% at the former).
bool cg_persist_plan(int num_cus, const Geom &g, int prec, int rows, PersistPlan &plan)
{
    if (prec != STAG_FP64 && prec != STAG_FP32_RU)
        return false;
    int lps = blocks_for_lps(g, 4) <= kFlatBlocks || (prec == STAG_FP64 && rows == 3) ? 4 : 2;
    if (const char *e = getenv("STAG_PERSIST")) {  // 0: never, 2 / 4: that many lanes per site
        const int v = atoi(e);
        if (v == 0)
            return false;
        if (v == 2 || v == 4)
            lps = v;
    }
    if (lps == 2 && prec == STAG_FP64 && rows == 3)
        return false;
    plan.lps = lps;
    plan.nblk = blocks_for_lps(g, lps);
    return plan.nblk <= std::min(num_cus, kMaxBlocks);
}

hipError_t cg_persist_launch(const PersistPlan &plan, int prec, int rows, const CgArgs &a, void *slots, uint32_t seq0,
                             int max_steps, hipStream_t s)
{
    PersistArgs pa;
    pa.c = a;
    pa.slots = (unsigned long long *)slots;
    pa.abort = (int *)((char *)slots + (size_t)(kBlockWords + kGroupWords) * 8);
    pa.seq0 = seq0;
    pa.max_steps = max_steps;
    pa.wait_ticks = kWaitTicks;
    if (const char *e = getenv("STAG_PERSIST_TICKS"))  // tests: 0 gives up at the first sum
        pa.wait_ticks = strtoull(e, nullptr, 10);
#define STAG_PERSIST_CASE(P, LPS)                                                                          \
    return rows == 2 ? launch<P, LPS, 2>(pa, plan.nblk, s) : launch<P, LPS, 3>(pa, plan.nblk, s)
    if (prec == STAG_FP64) {
        if (plan.lps == 4)
            STAG_PERSIST_CASE(PrecF64, 4);
        return rows == 2 ? launch<PrecF64, 2, 2>(pa, plan.nblk, s) : hipErrorInvalidValue;
    }
    if (plan.lps == 4)
        STAG_PERSIST_CASE(PrecF32, 4);
    STAG_PERSIST_CASE(PrecF32, 2);
#undef STAG_PERSIST_CASE
}

}  // namespace stag
