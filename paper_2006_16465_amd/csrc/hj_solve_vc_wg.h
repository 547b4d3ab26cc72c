// hj_solve_vc_wg.h -- whole variable-coefficient solves, one workgroup per
// right-hand side.
//
// A hierarchical cycle whose overlap reaches 2 s - 2 on each axis that has
// more than one tile gives every owned point the values of s sweeps of the
// whole grid, bit for bit (a frozen halo value reaches one point further into
// the tile per sweep after the first, and the tile hands over the points at
// least s away from it).  So on a grid whose points, right-hand side and face
// weights fit one workgroup's registers, the cycles are sweeps of the whole
// grid by that workgroup: no launch, no loads and no halo work between them (the
// iterate a cycle starts from is stored where it may be the one to stop at).  The residual of the iterate a cycle starts from is formed in
// its first sweep and judged before the next cycle, so the solve stops at the
// same iterate as the per-cycle path.
#pragma once

#include "hj_launch.h"
#include "hj_tiles.h"
#include "hj_wg.h"

namespace hj {
namespace {

constexpr int kVcWaves = 8;  // most wavefronts of a workgroup

// Rows that wavefronts hand to each other, by sweep parity.
struct VcWgLds {
    double bot[2][kVcWaves + 1][64];  // wavefront w's last row in [w + 1]; [0] is the boundary
    double top[2][kVcWaves + 1][64];  // wavefront w's first row in [w]; the one after the last is the boundary
    // Wavefront sums of one iterate's residual.  There is one set: between its
    // reading and the next posting every path has a barrier, of a sweep (the
    // first of the next cycle) or before the last iterate's residual.
    double red[kVcWaves];
};

// The value of the lane CTRL selects, 0 where there is none.
template <int CTRL>
__device__ __forceinline__ double dpp_edge0(double v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// Cycles [c_begin, c_end) of one solve (c_end <= maxc + 1; the pass for
// c == maxc runs no sweep, it only evaluates the residual of iterate maxc).
// u holds iterate c_begin on entry and on return the iterate the solve
// stopped at, or iterate c_end (c_end <= maxc) / maxc.  every: judge every
// iterate, else only iterates 0 and maxc.  A solve that has stopped returns at
// once.  MASK: the grid does not fill the workgroup's 64 columns and R rows a
// wavefront.
//
// Wavefront w holds rows [wR, wR + R), lane j column j of them: iterate, f,
// the weights of its west, east and north faces and 1 / (sum of the four),
// with the arithmetic of hj_vc_tile.h (whose values at every point it gives,
// so points off the grid are kept at zero, not only weighted with it: a value
// that is not finite must not come back over the boundary).
//
// What bounds it: FP64 issue, 13 instructions a point and sweep (nine of the
// update, four of the neighbour columns' DPP) at a wavefront instruction in
// four cycles.  Two wavefronts a SIMD hide the arithmetic's latency, and a
// wavefront of whole rows hands only its outer two to LDS, with R - 2 rows of
// work beside that way and the barrier.  16-lane row groups of four columns a
// lane, as in hj_vc_tile.h, need a quarter of the DPP but wait for the rows of
// every group: 4.8 us a cycle of 16 right-hand sides at 64 x 64, s = 8, in
// place of 3.8 (a launch per cycle: 11.3).
template <int R, bool MASK>
__device__ __forceinline__ void solve_vc_body(const GeomVC &g, const double *__restrict__ f, double *__restrict__ u,
                                              int s, int64_t c_begin, int64_t c_end, int64_t maxc, double tol,
                                              bool every, Ctrl *ctrl, VcWgLds &L)
{
    static_assert(R >= 2, "an outer row on either side");
    // Solve state, identical in every thread (read before any thread of this
    // launch writes the block: the writes below follow at least one barrier).
    WgJudge J;
    J.status = ctrl->status;
    if (every && J.status != ST_RUNNING) return;
    J.r0sq = ctrl->r0sq;
    J.last = ctrl->last_rsq;
    J.done = ctrl->done_cycle;
    J.tol = tol;
    J.set_lim();

    const int j = (int)threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nw = (int)blockDim.x >> 6;
    const int r0 = wave * R;
    const int64_t ld = g.ld;
    const int vr = MASK ? min(g.ny - r0, R) : R;  // the wavefront's rows on the grid
    auto on = [&](int i) { return !MASK || (i < vr && j < g.nx); };

    double x[R], fv[R], fw[R], fe[R], fn[R], di[R], fs0;
    {
        const double *ab = g.a + (int64_t)r0 * g.lda + j;  // the node up and left of the lane's first point
        double A[R + 2][3];
#pragma unroll
        for (int ii = 0; ii < R + 2; ++ii)
#pragma unroll
            for (int cc = 0; cc < 3; ++cc)
                A[ii][cc] = !MASK || (ii < vr + 2 && j < g.nx) ? ab[(int64_t)ii * g.lda + cc] : 0.0;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int64_t at = (int64_t)(r0 + i) * ld + j;
            x[i] = on(i) ? u[at] : 0.0;
            fv[i] = on(i) ? f[at] : 0.0;
            fw[i] = 0.5 * (A[i + 1][1] + A[i + 1][0]) * g.ihx2;
            fe[i] = 0.5 * (A[i + 1][1] + A[i + 1][2]) * g.ihx2;
            fn[i] = 0.5 * (A[i + 1][1] + A[i + 2][1]) * g.ihy2;
        }
        fs0 = 0.5 * (A[1][1] + A[0][1]) * g.ihy2;
#pragma unroll
        for (int i = 0; i < R; ++i) di[i] = 1.0 / ((fw[i] + fe[i]) + ((i > 0 ? fn[i - 1] : fs0) + fn[i]));
    }
    if (threadIdx.x < 64) {
        L.bot[0][0][j] = L.bot[1][0][j] = 0.0;
        L.top[0][nw][j] = L.top[1][nw][j] = 0.0;
    }
    if (threadIdx.x < kVcWaves) L.red[threadIdx.x] = 0.0;

    // Rows beside the lane's, for the next sweep; par: the buffer they came
    // from.  A buffer is rewritten two sweeps later, after a barrier every
    // thread reaches only once its reads from it are done.
    double up, dn;
    int par = 0;
    auto publish = [&](double first, double last) {
        L.top[par][wave][j] = first;
        L.bot[par][wave + 1][j] = last;
    };
    auto fetch = [&]() {
        up = L.bot[par][wave][j];
        dn = L.top[par][wave + 1][j];
    };
    // new value of the point in row i from its old value xi and the old rows
    // above and below; RES: its part of the old iterate's squared residual
    // norm onto rsq
    auto point = [&]<bool RES>(int i, double xi, double us, double un, double &rsq) {
        const double uw = dpp_edge0<kDppWaveShr1>(xi), ue = dpp_edge0<kDppWaveShl1>(xi);
        const double sf = i > 0 ? fn[i - 1] : fs0;
        if (RES) {
            const double ax = (fw[i] * (xi - uw) + fe[i] * (xi - ue)) + (sf * (xi - us) + fn[i] * (xi - un));
            const double rr = on(i) ? fv[i] - ax : 0.0;
            rsq = __builtin_fma(rr, rr, rsq);
        }
        const double v = (fv[i] + ((fw[i] * uw + fe[i] * ue) + (sf * us + fn[i] * un))) * di[i];
        return on(i) ? v : 0.0;
    };
    // One sweep: the outer rows, which the neighbours wait for, then the inner
    // ones on both sides of the barrier, so that neither the way of the outer
    // rows through LDS nor the barrier is waited for.  mid: runs just before
    // the barrier, after: behind it.
    auto sweep = [&]<bool RES>(auto mid, auto after) {
        double rsq = 0.0;
        const double n0 = point.template operator()<RES>(0, x[0], up, x[1], rsq);
        const double nl = point.template operator()<RES>(R - 1, x[R - 1], x[R - 2], dn, rsq);
        par ^= 1;
        publish(n0, nl);
        __builtin_amdgcn_sched_barrier(0);
        double prev = x[0];
        auto inner = [&](int i) {
            const double v = point.template operator()<RES>(i, x[i], prev, x[i + 1], rsq);
            prev = x[i];
            x[i] = v;
        };
#pragma unroll
        for (int i = 1; i < R / 2; ++i) inner(i);
        mid();
        __syncthreads();
        fetch();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = R / 2; i < R - 1; ++i) inner(i);
        after();
        x[R - 1] = nl;
        x[0] = n0;
        return rsq;
    };
    auto none = [] {};
    auto post = [&](double sum) {
        if (j == 63) L.red[wave] = sum;
    };
    auto store = [&]() {
#pragma unroll
        for (int i = 0; i < R; ++i)
            if (on(i)) u[(int64_t)(r0 + i) * ld + j] = x[i];
    };
    auto leave = [&](int64_t c) {
        if (threadIdx.x == 0) {
            ctrl->r0sq = J.r0sq;
            ctrl->last_rsq = J.last;
            ctrl->iter = c;
            ctrl->done_cycle = J.done;
            ctrl->status = J.status;
        }
    };

    publish(x[0], x[R - 1]);
    __syncthreads();
    fetch();
    const int64_t c_sweep = c_end < maxc ? c_end : maxc;  // cycles with sweeps: [c_begin, c_sweep)
    for (int64_t c = c_begin; c < c_sweep; ++c) {
        // iterate c, in case the verdict on it is to stop here
        if (every && c > c_begin) store();
        double tot = 0.0;
        const double mine = sweep.template operator()<true>(none, none);
        if (s > 1) {
            sweep.template operator()<false>([&] { post(wave_sum63(mine)); }, [&] { tot = tree_sum<kVcWaves>(L.red); });
        } else {
            post(wave_sum63(mine));
            __syncthreads();
            tot = tree_sum<kVcWaves>(L.red);
        }
        // two sweeps a trip: they trade the rows' registers
        int it = 2;
        for (; it + 1 < s; it += 2) {
            sweep.template operator()<false>(none, none);
            sweep.template operator()<false>(none, none);
        }
        if (it < s) sweep.template operator()<false>(none, none);
        // the verdict on iterate c
        if (every && J.far(tot)) {
            J.last = tot;
        } else if (every || c == 0) {
            J.take(c, tot);
            if (every && J.status != ST_RUNNING) {
                leave(c);
                return;
            }
        }
    }
    store();
    if (c_end == maxc + 1) {
        // with s <= 2 no barrier has followed the reading of iterate maxc - 1's
        // sums: a wavefront that posted now would change them under a later one
        __syncthreads();
        double rsq = 0.0;
#pragma unroll
        for (int i = 0; i < R; ++i)
            point.template operator()<true>(i, x[i], i > 0 ? x[i - 1] : up, i < R - 1 ? x[i + 1] : dn, rsq);
        post(wave_sum63(rsq));
        __syncthreads();
        J.take(maxc, tree_sum<kVcWaves>(L.red));
    }
    leave(c_sweep);
}

// Workgroup b solves right-hand side b; launched with the wavefronts that hold
// the grid's rows.
template <int R, bool MASK>
__global__ __launch_bounds__(64 * kVcWaves) void k_solve_vc_wg(GeomVC g, const double *__restrict__ f,
                                                         double *__restrict__ u, int64_t stride, int s,
                                                         int64_t c_begin, int64_t c_end, int64_t maxc, double tol,
                                                         int every, Ctrl *ctrls)
{
    __shared__ VcWgLds L;
    const int64_t b = blockIdx.x;
    solve_vc_body<R, MASK>(g, f + b * stride, u + b * stride, s, c_begin, c_end, maxc, tol, every != 0,
                                    ctrls + b, L);
}

}  // namespace
}  // namespace hj
