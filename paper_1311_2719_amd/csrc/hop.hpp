// The staggered hop sum (the inner loop of the paper's matrix-vector routine,
// Sec. 3) as device building blocks shared by the standalone D_slash and the
// fused CG kernels.
//
// One output site is processed by LPS lanes (LPS = 1, 2, 4, 8) of one
// wavefront.  Lanes are numbered sub-major: lane = sub * (64/LPS) + i, so the
// lanes that share `sub` take 64/LPS consecutive sites and every load they
// issue is unit-stride.  Lane `sub` takes mu = sub, sub + LPS, ..., forward
// and backward (LPS = 8: one of the eight hops), and the partial sums of a
// site are combined with cross-lane shuffles (xor 32, 16, 8).  R right-hand sides that share the gauge field are processed
// together so that each link entry is loaded once for all of them.
#pragma once

#include "stag_types.hpp"

namespace stag {

// Map the hardware block index to a logical one so that each XCD (blocks are
// dealt to the 8 XCDs round-robin) works on one contiguous range of sites:
// neighbour spinors of a range then stay in that XCD's L2.
__device__ __forceinline__ int logical_block(int b, int nblocks, int remap)
{
    if (!remap)
        return b;
    const int q = nblocks >> 3, rem = nblocks & 7;
    const int xcd = b & 7, i = b >> 3;
    return xcd * q + (xcd < rem ? xcd : rem) + i;
}

// Chunk of sites and tile (right-hand sides of one output parity) of this
// block, in a one-dimensional grid of chunks x ntiles blocks.  remap 1: each
// XCD takes one contiguous range of chunks and all tiles of a chunk follow one
// another: the two parities' tiles, which use the same links from their two
// ends, then find them in that XCD's L2 (FP64 32^4: 103 us interleaved, 152 us
// and two copies of the links before).  remap 2: one tile after the other, each
// XCD on one contiguous range of each (batched tiles, whose vectors need the
// L2 more than the links do).  remap 3: as 1, but each XCD sweeps its eighth of
// the chunks of every t-slice (slice_chunks, a multiple of 8) through t, so
// that a site's t-neighbours were visited one eighth of a slice before and are
// still in the L2 (FP32 and FP16 at 32^4 5 to 10% per step, FP64 at 24^4 15%;
// FP64 at 32^4 loses 8%: an eighth of a slice there exceeds the 4 MB).  remap
// 0: one tile after the other, blocks dealt to the XCDs in turn.
struct BlockTile {
    int chunk, nchunks, tile;
};

__device__ __forceinline__ BlockTile block_tile(int ntiles, int remap, int slice_chunks)
{
    const int nch = (int)gridDim.x / ntiles, b = (int)blockIdx.x;
    if (remap == 1) {
        const int l = logical_block(b, gridDim.x, 1);
        return {l / ntiles, nch, l % ntiles};
    }
    if (remap == 3) {
        const int i = b >> 3, q = i / ntiles, w = slice_chunks >> 3;
        return {(q / w) * slice_chunks + (b & 7) * w + q % w, nch, i % ntiles};
    }
    return {logical_block(b % nch, nch, remap), nch, b / nch};
}

// Whether a grid of `nch` chunks of `block` threads, lps lanes per site, may
// use remap 3: whole chunks per t-slice, eight or a multiple, each visited once.
inline bool slices_divide(const Geom &g, int lps, int block, int64_t nch)
{
    const int64_t t = (int64_t)g.st * lps;
    return t % block == 0 && t / block % 8 == 0 && nch * block == (int64_t)g.Vh * lps;
}

// Site and lane-within-site of global thread gt (blocks are whole wavefronts).
template <int LPS> __device__ __forceinline__ void site_of_thread(int gt, int &s, int &sub)
{
    constexpr int SPW = 64 / LPS;  // sites per wavefront
    const int lane = gt & 63;
    sub = lane / SPW;
    s = (gt >> 6) * SPW + (lane % SPW);
}

template <int LPS, typename T> __device__ __forceinline__ T lane_sum(T v)
{
#pragma unroll
    for (int o = 32; o >= 64 / LPS; o >>= 1)
        v += __shfl_xor(v, o);
    return v;
}

// Entries of the link at lp (rows 0 and 1 and, with ROWS = 3, row 2).
template <class P, int ROWS, bool BACK>
__device__ __forceinline__ void load_link_rows(const typename P::link_t *lp, cplx<typename P::real> (&U)[9])
{
#pragma unroll
    for (int k = 0; k < 3 * ROWS; ++k)
        U[k] = BACK ? P::load_back_link(lp + k * kLinkTile) : P::load_link(lp + k * kLinkTile);
}

// acc[r][a] += sum over this lane's hops at output site s of parity p_out (see
// the layout in stag_types.hpp; lout / lin: the links of the output parity and
// of the other one), then summed over the LPS lanes of the site.  load(r, n, chi)
// fetches the
// input colour vector of right-hand side r at neighbour site n.  Every
// right-hand side of the tile is computed, so load must stay in bounds for
// each r; callers discard the sums of systems they do not update (a
// per-system test inside the direction loop would split it into blocks that
// each wait for their loads).  LEAN keeps
// the direction loop rolled (one mu, two directions' loads in flight at a
// time), for rarely taken paths that must not raise the register budget of
// the kernel they live in.  ROWS = 3: all 9 link entries are stored; ROWS = 2:
// rows 0 and 1 are stored and row 2 is rebuilt in registers.
template <class P, int LPS, int R, class Load, bool LEAN, int ROWS, bool TABLES>
__device__ __forceinline__ void hop_accumulate_impl(const Geom &g, const typename P::link_t *__restrict__ lout,
                                                    const typename P::link_t *__restrict__ lin,
                                                    const int32_t *__restrict__ nbr, int p_out, int s, int sub,
                                                    cplx<typename P::real> (*acc)[3], Load load)
{
    using real = typename P::real;
    static_assert(ROWS == 2 || ROWS == 3, "links are stored with 2 or 3 rows");
    SiteCoord c;
    if constexpr (!TABLES || ROWS == 2)
        c = decode_site(g, p_out, s);
    auto neighbour_of = [&](int d) {
        if constexpr (TABLES)
            return nbr[(int64_t)d * g.Vh + s];
        else
            return neighbour(g, c, s, d);
    };
    auto forward = [&](int mu) {
        const int n = neighbour_of(mu);
        cplx<real> U[9];
        load_link_rows<P, ROWS, false>(lout + link_offset(ROWS, mu, s), U);
        if constexpr (ROWS == 2)
            third_row(U, folded_negative(g, c, mu) ? real(-2) : real(2));
#pragma unroll
        for (int r = 0; r < R; ++r) {
            cplx<real> chi[3];
            load(r, n, chi);
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int b = 0; b < 3; ++b)
                    cmac(acc[r][a], U[a * 3 + b], chi[b]);
        }
    };
    auto backward = [&](int mu) {
        const int n = neighbour_of(4 + mu);
        cplx<real> U[9];
        load_link_rows<P, ROWS, true>(lin + link_offset(ROWS, mu, n), U);
        if constexpr (ROWS == 2)
            third_row(U, folded_negative(g, c, 4 + mu) ? real(2) : real(-2));
#pragma unroll
        for (int r = 0; r < R; ++r) {
            cplx<real> chi[3];
            load(r, n, chi);
#pragma unroll
            for (int b = 0; b < 3; ++b)
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    cmsub_conj(acc[r][a], U[b * 3 + a], chi[b]);
        }
    };
    if constexpr (LPS == 8) {
        // one hop per lane, forward or backward by lane: the matrix is formed
        // by selects, so the lanes of a wavefront do not diverge
        const int mu = sub & 3;
        const bool back = sub >= 4;
        const int n = neighbour_of(sub);
        cplx<real> U[9];
        load_link_rows<P, ROWS, false>((back ? lin : lout) + link_offset(ROWS, mu, back ? n : s), U);
        if constexpr (ROWS == 2)
            third_row(U, folded_negative(g, c, sub) != back ? real(-2) : real(2));
        cplx<real> M[9];
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const cplx<real> u = U[a * 3 + b], v = U[b * 3 + a];
                M[a * 3 + b] = {back ? -v.re : u.re, back ? v.im : u.im};
            }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            cplx<real> chi[3];
            load(r, n, chi);
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int b = 0; b < 3; ++b)
                    cmac(acc[r][a], M[a * 3 + b], chi[b]);
        }
    } else if constexpr (LEAN) {
#pragma unroll 1
        for (int j = 0; j < 4 / LPS; ++j) {
            forward(sub + j * LPS);
            backward(sub + j * LPS);
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4 / LPS; ++j) {
            forward(sub + j * LPS);
            backward(sub + j * LPS);
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            acc[r][a].re = lane_sum<LPS>(acc[r][a].re);
            acc[r][a].im = lane_sum<LPS>(acc[r][a].im);
        }
}

// The hop with the neighbour source (tables or coordinates) decided once,
// outside the direction loop: a choice inside it would merge the table load
// and the computed index into one register, and the wait for that load would
// drain every load in flight at each direction.
template <class P, int LPS, int R, class Load, bool LEAN = false, int ROWS = 3>
__device__ __forceinline__ void hop_accumulate(const Geom &g, const typename P::link_t *__restrict__ lout,
                                               const typename P::link_t *__restrict__ lin,
                                               const int32_t *__restrict__ nbr, int p_out, int s, int sub,
                                               cplx<typename P::real> (*acc)[3], Load load)
{
    if (nbr)
        hop_accumulate_impl<P, LPS, R, Load, LEAN, ROWS, true>(g, lout, lin, nbr, p_out, s, sub, acc, load);
    else
        hop_accumulate_impl<P, LPS, R, Load, LEAN, ROWS, false>(g, lout, lin, nbr, p_out, s, sub, acc, load);
}

// Colour c of an output site is written / reduced by lane (c mod LPS).
template <int LPS> __device__ __forceinline__ bool owns_colour(int sub, int c) { return (c % LPS) == sub; }

// ---- block reductions (deterministic: fixed shuffle tree, fixed LDS order) ----

// A double moved across lanes by a DPP control (two 32-bit moves).
template <int CTRL> __device__ __forceinline__ double dpp_move(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ double read_lane(double v, int lane)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), lane);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Sum over the 64 lanes of a wavefront (every lane must be active), returned
// in every lane.  Within each row of 16 lanes the sum is formed by DPP moves
// (pairs, quads, half-row mirror, row mirror: no LDS round trips), then the
// four row sums are added in a fixed order.
__device__ __forceinline__ double wave_sum(double v)
{
    v += dpp_move<0xb1>(v);   // quad_perm [1,0,3,2]
    v += dpp_move<0x4e>(v);   // quad_perm [2,3,0,1]
    v += dpp_move<0x141>(v);  // row_half_mirror
    v += dpp_move<0x140>(v);  // row_mirror
    return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}

// Sum v[r] over the block; thread r (< R) receives the total of column r.
// lds must hold R * (blockDim.x / 64) doubles.
template <int R> __device__ __forceinline__ void block_sum_multi(double (&v)[R], double *lds, double &out)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const double t = wave_sum(v[r]);
        if (lane == 0)
            lds[r * nw + w] = t;
    }
    __syncthreads();
    out = 0.0;
    if (threadIdx.x < R)
        for (int i = 0; i < nw; ++i)
            out += lds[threadIdx.x * nw + i];
    __syncthreads();
}

// Total of partials[0 .. n) in a fixed order (a strided sum per thread, then
// the block tree); valid in thread 0.
__device__ __forceinline__ double reduce_partials(const double *partials, int n, double *lds)
{
    double v = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x)
        v += partials[i];
    double arr[1] = {v};
    double out;
    block_sum_multi<1>(arr, lds, out);
    return out;
}

}  // namespace stag
