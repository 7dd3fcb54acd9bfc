// Gauge-field preparation (the role of the paper's `linkc_acc`, Sec. 4) and
// fermion layout conversion.
//
// From lexicographic links U_mu(x) (complex128 [V][4][3][3]) build, for each
// parity p and checkerboard site s of it, the four forward links
//   W_mu(x) = 1/2 eta_mu(x) s(x, mu) U_mu(x),
// s = -1 on the hop from t = Lt-1 to t = 0 when the field is antiperiodic in t.
// The paper also gathers ud = U^dagger through the backward neighbour table; a
// hop here daggers the neighbour's W_mu in registers (eta_mu(x - mu) =
// eta_mu(x), because eta_mu does not depend on x_mu), so no second copy is
// kept.  When every one of these matrices is 1/2 (with a sign) times a special
// unitary matrix, only their first two rows are stored and the kernels rebuild
// the third (two-row form, 2/3 of the link bytes).
#include <cstdlib>

#include "runtime.hpp"

namespace stag {

namespace {

// The forward link mu of checkerboard site s of parity p with the folded
// factor (see above): w[k] = entry k (row-major) of W_mu(x).  Returns false if
// an entry is not finite.
__device__ bool folded_link(const Geom &g, const double *__restrict__ U, int p, int mu, int s, dbl2 (&w)[9])
{
    const SiteCoord c = decode_site(g, p, s);
    const double fac = folded_negative(g, c, mu) ? -0.5 : 0.5;
    const int64_t lex = c.x + (int64_t)g.L[0] * (c.y + (int64_t)g.L[1] * (c.z + (int64_t)g.L[2] * c.t));
    const double *u = U + (lex * 4 + mu) * 18;
    bool finite = true;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const double re = u[2 * k], im = u[2 * k + 1];
        w[k] = dbl2{re * fac, im * fac};
        finite = finite && isfinite(re) && isfinite(im);
    }
    return finite;
}

// flags |= 1 if any entry is not finite; |= 2 if some stored matrix is not
// (1/2 sign) x a special unitary matrix to within `tol` in the sense the
// two-row form relies on: row 2 = conj(row 0 x row 1) / c.
__global__ void __launch_bounds__(256)
k_check_links(Geom g, const double *__restrict__ U, double tol, int *__restrict__ flags)
{
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= (int64_t)2 * 4 * g.Vh)
        return;
    const int s = (int)(gid % g.Vh);
    const int mu = (int)((gid / g.Vh) % 4);
    const int p = (int)(gid / ((int64_t)4 * g.Vh));
    dbl2 w[9];
    int f = 0;
    if (!folded_link(g, U, p, mu, s, w)) {
        f = 1;
    } else {
        cplx<double> W[9];
        for (int k = 0; k < 9; ++k)
            W[k] = {w[k].x, w[k].y};
        const cplx<double> given[3] = {W[6], W[7], W[8]};
        third_row(W, folded_negative(g, decode_site(g, p, s), mu) ? -2.0 : 2.0);
        double dev = 0.0;
        for (int k = 0; k < 3; ++k)
            dev = fmax(dev, fmax(fabs(W[6 + k].re - given[k].re), fabs(W[6 + k].im - given[k].im)));
        if (!(dev <= tol))
            f = 2;
    }
    if (f)
        atomicOr(flags, f);
}

// Write the 3 * ROWS stored entries of every link in FP64, FP32 and FP16, and
// the neighbour tables.
template <int ROWS>
__global__ void __launch_bounds__(256)
k_prepare_links(Geom g, const double *__restrict__ U, dbl2 *__restrict__ l64, flt2 *__restrict__ l32,
                hlf2 *__restrict__ l16, int32_t *__restrict__ nbr)
{
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= (int64_t)2 * 4 * g.Vh)
        return;
    const int s = (int)(gid % g.Vh);
    const int mu = (int)((gid / g.Vh) % 4);
    const int p = (int)(gid / ((int64_t)4 * g.Vh));
    dbl2 w[9];
    (void)folded_link(g, U, p, mu, s, w);
    const int64_t base = link_parity_entries(ROWS, g.Vh) * p + link_offset(ROWS, mu, s);
#pragma unroll
    for (int k = 0; k < 3 * ROWS; ++k) {
        const int64_t o = base + k * kLinkTile;
        l64[o] = w[k];
        l32[o] = flt2{(float)w[k].x, (float)w[k].y};
        l16[o] = hlf2{(_Float16)w[k].x, (_Float16)w[k].y};
    }
    const SiteCoord c = decode_site(g, p, s);
    nbr[((int64_t)p * 8 + mu) * g.Vh + s] = neighbour(g, c, s, mu);
    nbr[((int64_t)p * 8 + 4 + mu) * g.Vh + s] = neighbour(g, c, s, 4 + mu);
}

// lexicographic [V][3] <-> even-odd [2][3][Vh]
__global__ void __launch_bounds__(256)
k_pack(Geom g, dbl2 *__restrict__ lex, dbl2 *__restrict__ eo, int to_eo)
{
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= (int64_t)2 * g.Vh)
        return;
    const int p = (int)(gid / g.Vh);
    const int s = (int)(gid % g.Vh);
    const SiteCoord c = decode_site(g, p, s);
    const int64_t l = c.x + (int64_t)g.L[0] * (c.y + (int64_t)g.L[1] * (c.z + (int64_t)g.L[2] * c.t));
#pragma unroll
    for (int col = 0; col < 3; ++col) {
        const int64_t e = ((int64_t)p * 3 + col) * g.Vh + s;
        if (to_eo)
            eo[e] = lex[l * 3 + col];
        else
            lex[l * 3 + col] = eo[e];
    }
}

}  // namespace

void choose_link_loads(GaugeField &f)
{
    if (const char *e = getenv("STAG_NT_LINKS"))
        if (e[0] == '0' || e[0] == '1') {
            f.nt_links = f.nt_once = e[0] == '1';
            return;
        }
    const size_t fp64_link_bytes = (size_t)2 * link_parity_entries(f.rows, f.g.Vh) * link_entry_bytes_of(0);
    f.nt_links = fp64_link_bytes > ((size_t)256 << 20);
    // between 128 and 256 MiB: a hop of one parity on one field after another
    // 53.4 us with plain loads, 49.7 without keeping the lines (28^4; the one
    // field repeated 42 and 49); both parities and the solves keep plain ones
    f.nt_once = fp64_link_bytes > ((size_t)128 << 20);
}

int gauge_check(Ctx *ctx, const Geom &g, const double *links_dev, hipStream_t s, bool &two_rows)
{
    const int64_t n = (int64_t)2 * 4 * g.Vh;
    int *flags = (int *)ctx->arena.alloc(256);
    if (!flags)
        return set_error(STAG_ENOMEM, "arena exhausted (gauge check flags)");
    int hflags = 0;
    hipError_t e = hipMemsetAsync(flags, 0, sizeof(int), s);
    if (e == hipSuccess) {
        const int threads = 256;
        hipLaunchKernelGGL(k_check_links, dim3((unsigned)((n + threads - 1) / threads)), dim3(threads), 0, s, g,
                           links_dev, kTwoRowTolerance, flags);
        e = hipGetLastError();
    }
    if (e == hipSuccess)
        e = hipMemcpyAsync(&hflags, flags, sizeof(int), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess)
        e = hipStreamSynchronize(s);
    ctx->arena.release(flags);
    if (e != hipSuccess)
        return set_error(STAG_EHIP, "gauge check failed: %s", hipGetErrorString(e));
    if (hflags & 1)
        return set_error(STAG_ENONFINITE, "gauge field holds NaN or Inf");
    two_rows = (hflags & 2) == 0;
    return STAG_OK;
}

int gauge_prepare(GaugeField *f, const double *links_dev, hipStream_t s)
{
    const Geom &g = f->g;
    const int64_t n = (int64_t)2 * 4 * g.Vh;
    const int threads = 256;
    const dim3 grid((unsigned)((n + threads - 1) / threads));
    if (f->rows == 2)
        hipLaunchKernelGGL((k_prepare_links<2>), grid, dim3(threads), 0, s, g, links_dev, (dbl2 *)f->links[0],
                           (flt2 *)f->links[1], (hlf2 *)f->links[2], f->nbr);
    else
        hipLaunchKernelGGL((k_prepare_links<3>), grid, dim3(threads), 0, s, g, links_dev, (dbl2 *)f->links[0],
                           (flt2 *)f->links[1], (hlf2 *)f->links[2], f->nbr);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess)
        e = hipStreamSynchronize(s);
    if (e != hipSuccess)
        return set_error(STAG_EHIP, "gauge preparation failed: %s", hipGetErrorString(e));
    return STAG_OK;
}

int launch_pack(const Geom &g, const double *lex, double *eo, int to_eo, hipStream_t s)
{
    const int threads = 256;
    const int64_t n = (int64_t)2 * g.Vh;
    const int64_t blocks = (n + threads - 1) / threads;
    hipLaunchKernelGGL(k_pack, dim3((unsigned)blocks), dim3(threads), 0, s, g,
                       (dbl2 *)const_cast<double *>(lex), (dbl2 *)eo, to_eo);
    STAG_HIP_CHECK(hipGetLastError());
    return STAG_OK;
}

}  // namespace stag
