// The standalone D_slash (the paper's matrix-vector routine of Sec. 3,
// `matrix-vector(offset, local_length, v, w)`, restricted to one parity or
// applied to the whole lattice) in FP64, FP32 or FP16, conversion of fermion
// fields between those storage precisions, and the kernel-configuration tuner.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "cg_launch.hpp"
#include "runtime.hpp"

namespace stag {

const CgLaunchTable &cg_table_f64();
const CgLaunchTable &cg_table_f32();
const CgLaunchTable &cg_table_f16();
const CgLaunchTable &cg_table_f64_r2();
const CgLaunchTable &cg_table_f32_r2();
const CgLaunchTable &cg_table_f16_r2();
const CgLaunchTable &cg_table_f64nt();
const CgLaunchTable &cg_table_f64nt_r2();

const CgLaunchTable &cg_table(int prec, int rows, int nt_links)
{
    if (prec == 0 && nt_links)
        return rows == 2 ? cg_table_f64nt_r2() : cg_table_f64nt();
    if (rows == 2)
        return prec == 0 ? cg_table_f64_r2() : prec == 1 ? cg_table_f32_r2() : cg_table_f16_r2();
    return prec == 0 ? cg_table_f64() : prec == 1 ? cg_table_f32() : cg_table_f16();
}

namespace {

// out(x) (+)= (D in)(x) for checkerboard sites [offset, offset + count) of the
// output parity (both parities, their blocks alternating, when par_fixed < 0), with
// links, vectors and arithmetic of precision P: FP64 / FP32 vectors are
// [parity][colour][Vh] complex, FP16 vectors [parity][Vh] records of three
// scaled half2 colours and their FP32 scale.
template <class P, int LPS, int ROWS>
__global__ void __launch_bounds__(256)
k_dslash(Geom g, const typename P::link_t *__restrict__ links, const int32_t *__restrict__ nbr,
         const void *__restrict__ in, void *__restrict__ out, int par_fixed, int offset, int count, int accumulate,
         int remap)
{
    using real = typename P::real;
    const BlockTile tl = block_tile(par_fixed >= 0 ? 1 : 2, remap, g.st * LPS / (int)blockDim.x);
    const int p = par_fixed >= 0 ? par_fixed : tl.tile;
    const int Vh = g.Vh;
    int site, sub;
    site_of_thread<LPS>(tl.chunk * blockDim.x + threadIdx.x, site, sub);
    if (site >= count)
        return;
    const int s = offset + site;
    const size_t half = (size_t)Vh * P::spinor_bytes;  // bytes of one parity half
    const char *src = (const char *)in + (size_t)(1 - p) * half;
    cplx<real> acc[1][3] = {{czero<real>(), czero<real>(), czero<real>()}};
    auto load = [&](int, int n, cplx<real> *chi) { P::load_spinor(src, Vh, n, chi); };
    const int64_t lp = link_parity_entries(ROWS, Vh);
    hop_accumulate<P, LPS, 1, decltype(load), false, ROWS>(g, links + lp * p, links + lp * (1 - p),
                                                           nbr ? nbr + (size_t)p * 8 * Vh : nullptr, p, s, sub, acc,
                                                           load);
    char *o = (char *)out + (size_t)p * half;
    if constexpr (P::id == 2) {
        // one lane writes the whole record (every lane holds the lane sum)
        if (sub != 0)
            return;
        if (accumulate) {
            cplx<real> old[3];
            P::load_spinor(o, Vh, s, old);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                acc[0][c].re += old[c].re;
                acc[0][c].im += old[c].im;
            }
        }
        P::store_spinor(o, Vh, s, acc[0]);
    } else {
        using v2 = typename vec2_of<real>::type;
        v2 *ov = (v2 *)o;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            if (!owns_colour<LPS>(sub, c))
                continue;
            v2 v = v2{acc[0][c].re, acc[0][c].im};
            if (accumulate)
                v += ov[(int64_t)c * Vh + s];
            ov[(int64_t)c * Vh + s] = v;
        }
    }
}

// Convert a full-lattice field (both parities, 2 Vh sites) between vector
// storage precisions: FP64 / FP32 [parity][colour][Vh] complex, FP16
// [parity][Vh] records.  One thread per site.
template <class PI, class PO>
__global__ void __launch_bounds__(256) k_convert(int Vh, const void *__restrict__ in, void *__restrict__ out)
{
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= (int64_t)2 * Vh)
        return;
    const int p = (int)(gid / Vh), s = (int)(gid % Vh);
    const char *ib = (const char *)in + (size_t)p * Vh * PI::spinor_bytes;
    char *ob = (char *)out + (size_t)p * Vh * PO::spinor_bytes;
    cplx<typename PI::real> v[3];
    PI::load_spinor(ib, Vh, s, v);
    cplx<typename PO::real> w[3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
        w[c] = {(typename PO::real)v[c].re, (typename PO::real)v[c].im};
    PO::store_spinor(ob, Vh, s, w);
}

template <class P>
hipError_t launch_dslash_p(const KernelCfg &cfg, const GaugeField *f, int par_fixed, int nparity, int offset,
                           int count, const void *in, void *out, int accumulate, hipStream_t s)
{
    const int64_t threads = (int64_t)count * cfg.lps;  // site = wave * (64/lps) + lane % (64/lps)
    dim3 grid((unsigned)((threads + cfg.block - 1) / cfg.block) * (unsigned)nparity);
    dim3 block(cfg.block);
    // t-columns need the whole parity; other site ranges take the XCD order
    const int remap = cfg.remap == 3 && !slices_divide(f->g, cfg.lps, cfg.block, grid.x / nparity) ? 1 : cfg.remap;
    const auto *lk = (const typename P::link_t *)f->links[P::id];
    const int32_t *nb = cfg.tables ? f->nbr : nullptr;
#define STAG_DSLASH_CASE(L, ROWS)                                                                                    \
    hipLaunchKernelGGL((k_dslash<P, L, ROWS>), grid, block, 0, s, f->g, lk, nb, in, out, par_fixed, offset, count,  \
                       accumulate, remap)
    const int key = cfg.lps * 4 + f->rows;
    switch (key) {
    case 1 * 4 + 3: STAG_DSLASH_CASE(1, 3); break;
    case 2 * 4 + 3: STAG_DSLASH_CASE(2, 3); break;
    case 4 * 4 + 3: STAG_DSLASH_CASE(4, 3); break;
    case 8 * 4 + 3: STAG_DSLASH_CASE(8, 3); break;
    case 1 * 4 + 2: STAG_DSLASH_CASE(1, 2); break;
    case 2 * 4 + 2: STAG_DSLASH_CASE(2, 2); break;
    case 4 * 4 + 2: STAG_DSLASH_CASE(4, 2); break;
    case 8 * 4 + 2: STAG_DSLASH_CASE(8, 2); break;
    default: return hipErrorInvalidValue;
    }
#undef STAG_DSLASH_CASE
    return hipGetLastError();
}

}  // namespace

int dslash(Ctx *ctx, GaugeField *f, int prec, int out_parity, int64_t offset, int64_t count, const void *in,
           void *out, int accumulate, hipStream_t s)
{
    return dslash_with(tune_config(ctx, f, prec, 1, out_parity != STAG_ALL, s), f, prec, out_parity, offset, count, in,
                       out, accumulate, s);
}

int dslash_with(const KernelCfg &cfg, GaugeField *f, int prec, int out_parity, int64_t offset, int64_t count,
                const void *in, void *out, int accumulate, hipStream_t s)
{
    const int Vh = f->g.Vh;
    const int par_fixed = out_parity == STAG_ALL ? -1 : out_parity;
    const int nparity = out_parity == STAG_ALL ? 2 : 1;
    const int off = out_parity == STAG_ALL ? 0 : (int)offset;
    const int cnt = out_parity == STAG_ALL ? Vh : (int)count;
    hipError_t e;
    switch (prec) {
    case 0:
        e = f->nt_once && nparity == 1
                ? launch_dslash_p<PrecF64NTOnce>(cfg, f, par_fixed, nparity, off, cnt, in, out, accumulate, s)
            : f->nt_links
                ? launch_dslash_p<PrecF64NT>(cfg, f, par_fixed, nparity, off, cnt, in, out, accumulate, s)
                : launch_dslash_p<PrecF64>(cfg, f, par_fixed, nparity, off, cnt, in, out, accumulate, s);
        break;
    case 1: e = launch_dslash_p<PrecF32>(cfg, f, par_fixed, nparity, off, cnt, in, out, accumulate, s); break;
    case 2: e = launch_dslash_p<PrecF16>(cfg, f, par_fixed, nparity, off, cnt, in, out, accumulate, s); break;
    default: return set_error(STAG_EINVAL, "dslash: unknown precision %d", prec);
    }
    if (e != hipSuccess)
        return set_error(STAG_EHIP, "dslash launch failed: %s", hipGetErrorString(e));
    return STAG_OK;
}

int dslash_f64(Ctx *ctx, GaugeField *f, int out_parity, int64_t offset, int64_t count, const double *in,
               double *out, int accumulate, hipStream_t s)
{
    return dslash(ctx, f, 0, out_parity, offset, count, in, out, accumulate, s);
}

int convert_fermion(const Geom &g, int prec_in, const void *in, int prec_out, void *out, hipStream_t s)
{
    const int64_t n = (int64_t)2 * g.Vh;
    dim3 grid((unsigned)((n + 255) / 256)), block(256);
#define STAG_CONVERT_CASE(PI, PO) hipLaunchKernelGGL((k_convert<PI, PO>), grid, block, 0, s, g.Vh, in, out)
    switch (prec_in * 3 + prec_out) {
    case 0: STAG_CONVERT_CASE(PrecF64, PrecF64); break;
    case 1: STAG_CONVERT_CASE(PrecF64, PrecF32); break;
    case 2: STAG_CONVERT_CASE(PrecF64, PrecF16); break;
    case 3: STAG_CONVERT_CASE(PrecF32, PrecF64); break;
    case 4: STAG_CONVERT_CASE(PrecF32, PrecF32); break;
    case 5: STAG_CONVERT_CASE(PrecF32, PrecF16); break;
    case 6: STAG_CONVERT_CASE(PrecF16, PrecF64); break;
    case 7: STAG_CONVERT_CASE(PrecF16, PrecF32); break;
    case 8: STAG_CONVERT_CASE(PrecF16, PrecF16); break;
    default: return set_error(STAG_EINVAL, "convert: unknown precision");
    }
#undef STAG_CONVERT_CASE
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return set_error(STAG_EHIP, "convert launch failed: %s", hipGetErrorString(e));
    return STAG_OK;
}

// ---- tuner ----------------------------------------------------------------------

static bool env_cfg(KernelCfg &c)
{
    const char *e = getenv("STAG_KERNEL_CFG");  // "lps,block,rtile,tables,remap"
    if (!e || !*e)
        return false;
    int v[5];
    if (sscanf(e, "%d,%d,%d,%d,%d", &v[0], &v[1], &v[2], &v[3], &v[4]) != 5)
        return false;
    c.lps = v[0];
    c.block = v[1];
    c.rtile = v[2];
    c.tables = v[3];
    c.remap = v[4];
    return true;
}

static bool valid_lps(int l) { return l == 1 || l == 2 || l == 4 || l == 8; }

static int default_rtile(const CgLaunchTable &t, int nrhs)
{
    int best = 1;
    for (int i = 0; i < t.n_rtiles; ++i)
        if (nrhs % t.rtiles[i] == 0)
            best = std::max(best, t.rtiles[i]);
    return best;
}

// Lanes per site of the D_slash by lattice size: more lanes where the sites
// alone leave the chip idle.  Fixed rather than timed, so that the order of a
// site's sum, and with it the last bits of D, never depends on a timing.
// Best of 24 shapes with 1 / 2 / 4 / 8 lanes, us: FP64 8^4 4.3 / 3.8 / 3.6 / 3.6, 12^3 16
// 4.6 / 4.4 / 4.5 / 5.1, 16^4 7.2 / 6.4 / 6.4 / 7.7, 32^4 106 / 102 / 110 / 109; FP32 8^4
// 4.1 / 3.7 / 3.5 / 3.6, 20^4 9.9 / 9.4 / 9.5 / 11.3, 32^4 42.5 / 41.9 / 47.5 / -; FP16
// 20^4 8.2 / 7.4 / 8.5 / 11.6, 32^4 27.5 / 28.0 / 35.5 / -.
static int dslash_lps(const GaugeField *f) { return 2 * (int64_t)f->g.Vh <= 20736 ? 4 : 2; }

static KernelCfg default_config(const GaugeField *f, int prec, int nrhs)
{
    KernelCfg best;
    best.lps = dslash_lps(f);
    best.block = 256;
    best.rtile = default_rtile(cg_table(prec, f->rows, f->nt_links), nrhs);
    best.tables = 0;
    best.remap = 1;
    return best;
}

// Key of the tuned D_slash shape: outputs of one parity are another kernel than
// outputs of both (other link loads, no link used twice) and have their own.
static uint64_t dslash_key(int prec, int nrhs, bool one_parity)
{
    return ((uint64_t)one_parity << 36) | ((uint64_t)prec << 32) | (uint32_t)nrhs;
}

KernelCfg cached_config(Ctx *ctx, GaugeField *f, int prec, int nrhs, bool one_parity)
{
    std::lock_guard<std::mutex> lk(ctx->mu);
    auto it = f->tuned.find(dslash_key(prec, nrhs, one_parity));
    return it != f->tuned.end() ? it->second : default_config(f, prec, nrhs);
}

KernelCfg tune_config(Ctx *ctx, GaugeField *f, int prec, int nrhs, bool one_parity, hipStream_t s)
{
    const uint64_t key = dslash_key(prec, nrhs, one_parity);
    {
        std::lock_guard<std::mutex> lk(ctx->mu);
        auto it = f->tuned.find(key);
        if (it != f->tuned.end())
            return it->second;
    }
    const CgLaunchTable &tab = cg_table(prec, f->rows, f->nt_links);
    KernelCfg best = default_config(f, prec, nrhs);
    KernelCfg forced;
    const char *tune_env = getenv("STAG_TUNE");
    const bool tune = !(tune_env && tune_env[0] == '0');
    if (env_cfg(forced)) {
        if (valid_lps(forced.lps) && forced.block >= 64 && forced.block <= 256 && forced.block % 64 == 0 &&
            nrhs % forced.rtile == 0)
            best = forced;
    } else if (tune) {
        // time out_r = D in_r on scratch vectors for every candidate; keep the
        // fastest per right-hand side
        std::vector<int> tiles;
        for (int i = 0; i < tab.n_rtiles; ++i)
            if (nrhs % tab.rtiles[i] == 0)
                tiles.push_back(tab.rtiles[i]);
        const bool verbose = getenv("STAG_TUNE_VERBOSE") != nullptr;
        // scratch vectors for every system of the solve shape (2 parities x nrhs)
        const size_t vbytes = (size_t)f->g.Vh * spinor_bytes_of(prec) * 2 * nrhs;
        void *in = ctx->arena.alloc(vbytes), *out = ctx->arena.alloc(vbytes);
        hipEvent_t e0 = nullptr, e1 = nullptr;
        bool ok = in && out && hipEventCreate(&e0) == hipSuccess && hipEventCreate(&e1) == hipSuccess &&
                  hipMemsetAsync(in, 0, vbytes, s) == hipSuccess;
        // one run of a shape, us per right-hand side (1e30: failed): the D_slash
        // itself for one right-hand side, else a probe of the tile
        auto timed = [&](const KernelCfg &c) {
            const int64_t threads = (int64_t)f->g.Vh * c.lps;
            const int ntiles = 2 * nrhs / c.rtile;
            dim3 grid((unsigned)((threads + c.block - 1) / c.block) * (unsigned)ntiles), block(c.block);
            const void *links = f->links_for(prec, 0);
            const int32_t *nb = c.tables ? f->nbr_for(0) : nullptr;
            auto run = [&]() {
                if (nrhs == 1)
                    return dslash_with(c, f, prec, one_parity ? STAG_EVEN : STAG_ALL, 0, f->g.Vh, in, out, 0, s) == STAG_OK;
                return tab.probe(c.lps, c.rtile, grid, block, s, f->g, links, nb, in, out, ntiles, c.remap) == hipSuccess;
            };
            if (!ok || !run()) {
                ok = false;
                return 1e30;
            }
            const int reps = tune_reps(f->g);
            (void)hipEventRecord(e0, s);
            for (int i = 0; i < reps; ++i)
                (void)run();
            (void)hipEventRecord(e1, s);
            ok = hipEventSynchronize(e1) == hipSuccess;
            float ms = 0.f;
            (void)hipEventElapsedTime(&ms, e0, e1);
            const double t = (double)ms * 1e3 / reps / nrhs;
            if (verbose)
                fprintf(stderr, "[stag tune] V=%d prec=%d nrhs=%d %s lps=%d block=%d rtile=%d tables=%d remap=%d: %.2f us "
                                "per rhs\n", 2 * f->g.Vh, prec, nrhs, one_parity ? "one parity" : "both parities", c.lps,
                        c.block, c.rtile, c.tables, c.remap, t);
            return ok ? t : 1e30;
        };
        // the block sizes and tiles, the block orders of the two best, and the
        // three best of all again and in turn (single runs vary by more than these
        // differ), then the tables where they gain
        struct Timed {
            KernelCfg c;
            double t;
        };
        std::vector<Timed> seen;
        auto by_time = [&] {
            std::stable_sort(seen.begin(), seen.end(), [](const Timed &x, const Timed &y) { return x.t < y.t; });
        };
        auto again = [&](size_t n) {
            for (int k = 0; k < 2; ++k)
                for (size_t i = 0; i < n && i < seen.size(); ++i)
                    seen[i].t = std::min(seen[i].t, timed(seen[i].c));
        };
        const int blk_c[3] = {64, 128, 256};
        for (int R : tiles)
            for (int B : blk_c) {
                KernelCfg c;
                c.lps = best.lps;
                c.block = B;
                c.rtile = R;
                seen.push_back({c, timed(c)});
            }
        by_time();
        for (size_t i = 0, n = std::min<size_t>(2, seen.size()); i < n; ++i)
            for (int X : {0, 2, 3}) {
                KernelCfg c = seen[i].c;
                c.remap = X;
                const int64_t threads = (int64_t)f->g.Vh * c.lps;
                if (X == 2 && one_parity)  // one tile: order 1
                    continue;
                if (X != 3 || slices_divide(f->g, c.lps, c.block, (threads + c.block - 1) / c.block))
                    seen.push_back({c, timed(c)});
            }
        by_time();
        again(3);
        by_time();
        if (ok && !seen.empty()) {
            best = seen[0].c;
            seen.resize(1);
            seen.push_back({best, 1e30});
            seen[1].c.tables = 1;
            again(2);
            if (seen[1].t < seen[0].t * 0.99)
                best.tables = 1;
        }
        if (e0)
            (void)hipEventDestroy(e0);
        if (e1)
            (void)hipEventDestroy(e1);
        ctx->arena.release(in);
        ctx->arena.release(out);
        (void)hipGetLastError();
    }
    std::lock_guard<std::mutex> lk(ctx->mu);
    f->tuned[key] = best;
    return best;
}

}  // namespace stag
