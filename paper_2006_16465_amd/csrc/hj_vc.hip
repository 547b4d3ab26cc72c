// hj_vc.hip -- variable-coefficient diffusion -div(a grad u) = f on the 2D
// grid: the hierarchical cycle, the residual, and the gradient of a loss with
// respect to the node coefficients a (adjoint face products).
//
// The operator, its face weights and the cycle body live in hj_vc_tile.h.
#include <hip/hip_runtime.h>

#include "hj_launch.h"
#include "hj_vc_tile.h"
#include "hj_solve_vc_wg.h"

namespace hj {
namespace {

template <int TX, int TY, bool RES, bool REG>
__global__ __launch_bounds__((vc_threads<TX, TY>()), (vc_min_waves<TX, REG>())) void k_cycle2d_vc(GeomVC g, const double *__restrict__ f,
                                                                    const double *__restrict__ xin,
                                                                    double *__restrict__ xout, int nsub,
                                                                    Red red, double tol)
{
    constexpr int NT = vc_threads<TX, TY>();
    if (RES && !judged_start<NT>(red, tol)) return;
    const int blk = judged_block<RES>();
    const double rsq = tile_vc<TX, TY, RES, REG>(g, xcd_tile(blk, judged_blocks<RES>()), f, xin, xout, nsub);
    if (RES) post_partial<NT>(rsq, &red.part_cur[blk]);
}

// classical sweep (SWEEP) and / or residual (RES; with r_out when !SWEEP)
template <bool RES, bool SWEEP>
__global__ __launch_bounds__(kNT) void k_sweep2d_vc(GeomVC g, const double *__restrict__ f,
                                                    const double *__restrict__ xin,
                                                    double *__restrict__ xout, Red red, double tol)
{
    constexpr bool judged = SWEEP && RES;
    if (judged && !judged_start<kNT>(red, tol)) return;
    const int blk = judged_block<judged>(), nblk = judged_blocks<judged>();
    const int64_t total = (int64_t)g.nx * g.ny;
    const int64_t i = (int64_t)xcd_tile(blk, nblk) * kNT + threadIdx.x;
    double rsq = 0.0;
    if (i < total) {
        const int r = (int)(i / g.nx), q = (int)(i - (int64_t)r * g.nx);
        const int64_t a = (int64_t)r * g.ld + q;
        const Face k = face_at(g, r, q);
        const double c = xin[a];
        const double uw = q > 0 ? xin[a - 1] : 0.0;
        const double ue = q + 1 < g.nx ? xin[a + 1] : 0.0;
        const double us = r > 0 ? xin[a - g.ld] : 0.0;
        const double un = r + 1 < g.ny ? xin[a + g.ld] : 0.0;
        if (SWEEP) xout[a] = (f[a] + ((k.w * uw + k.e * ue) + (k.s * us + k.n * un))) * k.dinv;
        if (RES) {
            const double rr = f[a] - ((k.w * (c - uw) + k.e * (c - ue)) + (k.s * (c - us) + k.n * (c - un)));
            if (!SWEEP && xout) xout[a] = rr;
            rsq += rr * rr;
        }
    }
    if (RES) post_partial<kNT>(rsq, &red.part_cur[blk]);
}

// dL/da at every node of the (ny+2) x (nx+2) grid, summed over nb right-hand
// sides: each face between nodes P and Q contributes
// -(1/2) (u_P - u_Q)(lam_P - lam_Q) / h^2 to both nodes (u = lam = 0 on the
// boundary).  Gathered per node, no atomics.
__global__ __launch_bounds__(kNT) void k_grad_a_vc(GeomVC g, const double *__restrict__ u,
                                                   const double *__restrict__ lam, int nb,
                                                   int64_t bstride, double *__restrict__ grad,
                                                   int64_t ldg)
{
    const int64_t total = (int64_t)(g.nx + 2) * (g.ny + 2);
    const int64_t i = (int64_t)blockIdx.x * kNT + threadIdx.x;
    if (i >= total) return;
    const int R = (int)(i / (g.nx + 2)), Q = (int)(i - (int64_t)R * (g.nx + 2));
    const int r = R - 1, q = Q - 1;  // interior coordinates of the node
    auto in = [&](int rr, int qq) { return rr >= 0 && rr < g.ny && qq >= 0 && qq < g.nx; };
    double acc = 0.0;
    for (int b = 0; b < nb; ++b) {
        const double *ub = u + (int64_t)b * bstride;
        const double *lb = lam + (int64_t)b * bstride;
        auto U = [&](int rr, int qq) { return in(rr, qq) ? ub[(int64_t)rr * g.ld + qq] : 0.0; };
        auto L = [&](int rr, int qq) { return in(rr, qq) ? lb[(int64_t)rr * g.ld + qq] : 0.0; };
        const double u0 = U(r, q), l0 = L(r, q);
        double t = 0.0;
        if (r >= 0 && r < g.ny) {  // x faces exist in interior rows
            if (q - 1 >= -1) t += (u0 - U(r, q - 1)) * (l0 - L(r, q - 1)) * g.ihx2;
            if (q + 1 <= g.nx) t += (u0 - U(r, q + 1)) * (l0 - L(r, q + 1)) * g.ihx2;
        }
        if (q >= 0 && q < g.nx) {  // y faces exist in interior columns
            if (r - 1 >= -1) t += (u0 - U(r - 1, q)) * (l0 - L(r - 1, q)) * g.ihy2;
            if (r + 1 <= g.ny) t += (u0 - U(r + 1, q)) * (l0 - L(r + 1, q)) * g.ihy2;
        }
        acc += -0.5 * t;
    }
    grad[(int64_t)R * ldg + Q] = acc;
}

template <int TX, int TY>
hipError_t cyc_vc(const GeomVC &g, int s, bool res, const double *f, const double *xin, double *xout,
                  const Red &red, double tol, hipStream_t st)
{
    const unsigned nb = (unsigned)cycle_vc_blocks(g) + (res ? 1 : 0);
    constexpr int NT = vc_threads<TX, TY>();
    static_assert(NT == 8 * TY, "cycle_vc_one_launch counts them so");
    if (!one_launch(nb, NT)) return hipErrorInvalidConfiguration;
    auto go = [&](auto kernel) {
        kernel<<<nb, NT, 0, st>>>(g, f, xin, xout, s, red, tol);
        return hipGetLastError();
    };
    if (vc_reg(g)) return res ? go(k_cycle2d_vc<TX, TY, true, true>) : go(k_cycle2d_vc<TX, TY, false, true>);
    return res ? go(k_cycle2d_vc<TX, TY, true, false>) : go(k_cycle2d_vc<TX, TY, false, false>);
}

template <int R>
hipError_t launch_vc_wg(const GeomVC &g, int64_t batch, int64_t stride, int s, const double *f, double *u,
                    int64_t c_begin, int64_t c_end, int64_t maxc, double tol, bool every, Ctrl *ctrls, hipStream_t st)
{
    const unsigned nw = (unsigned)(g.ny + R - 1) / R;
    auto go = [&](auto kernel) -> hipError_t {
        kernel<<<(unsigned)batch, 64 * nw, 0, st>>>(g, f, u, stride, s, c_begin, c_end, maxc, tol, every ? 1 : 0,
                                                    ctrls);
        return hipGetLastError();
    };
    if (g.nx == 64 && g.ny == (int)nw * R) return go(k_solve_vc_wg<R, false>);
    return go(k_solve_vc_wg<R, true>);
}

}  // namespace

bool cycle_vc_one_launch(const GeomVC &g) { return one_launch(cycle_vc_blocks(g) + 1, 8 * g.ty); }
int64_t sweep_vc_blocks(const GeomVC &g) { return ((int64_t)g.nx * g.ny + kNT - 1) / kNT; }

hipError_t launch_cycle_vc(const GeomVC &g, int s, bool res, const double *f, const double *xin,
                           double *xout, const Red &red, double tol, hipStream_t st)
{
#define HJ_TILE(a, b) \
    if (g.tx == a && g.ty == b) return cyc_vc<a, b>(g, s, res, f, xin, xout, red, tol, st);
    HJ_VC_TILES(HJ_TILE)
#undef HJ_TILE
    return hipErrorInvalidValue;
}

hipError_t launch_sweep_vc(const GeomVC &g, bool res, const double *f, const double *xin, double *xout,
                           const Red &red, double tol, hipStream_t st)
{
    const unsigned nb = (unsigned)sweep_vc_blocks(g) + (res ? 1 : 0);
    if (!one_launch(nb, kNT)) return hipErrorInvalidConfiguration;
    if (res) k_sweep2d_vc<true, true><<<nb, kNT, 0, st>>>(g, f, xin, xout, red, tol);
    else k_sweep2d_vc<false, true><<<nb, kNT, 0, st>>>(g, f, xin, xout, red, tol);
    return hipGetLastError();
}

hipError_t launch_resid_vc(const GeomVC &g, const double *f, const double *x, double *r_out,
                           double *part, hipStream_t st)
{
    const unsigned nb = (unsigned)sweep_vc_blocks(g);
    if (!one_launch(nb, kNT)) return hipErrorInvalidConfiguration;
    const Red red{part, nullptr, nullptr, 0, 0};
    k_sweep2d_vc<true, false><<<nb, kNT, 0, st>>>(g, f, x, r_out, red, -1.0);
    return hipGetLastError();
}

hipError_t launch_grad_a_vc(const GeomVC &g, const double *u, const double *lam, int nb,
                            int64_t bstride, double *grad, int64_t ldg, hipStream_t st)
{
    const int64_t total = (int64_t)(g.nx + 2) * (g.ny + 2), nb64 = (total + kNT - 1) / kNT;
    if (!one_launch(nb64, kNT)) return hipErrorInvalidConfiguration;
    k_grad_a_vc<<<(unsigned)nb64, kNT, 0, st>>>(g, u, lam, nb, bstride, grad, ldg);
    return hipGetLastError();
}

// Grids of at most 64 x 64 points whose cycle is s sweeps of the whole grid.
// There a sweep by one workgroup (0.38 us at 64 x 64) takes no longer than one
// by the workgroup of a 64 x 64 tile, and the cycle's launch, its loads and
// stores and the tiles' overlap fall away: us a cycle with a launch each and
// here, s = 8, overlap 14: one right-hand side at 64 x 64 (64 x 32 tiles) 7.8
// and 3.8, 16 of them 11.3 and 3.8, 1024 of them 48 and 17; four at 20 x 20
// (32 x 32 tiles) 11.4 and 2.5; 1024 at 30 x 30 20 and 8.9.  Higher grids do
// not fit a SIMD's registers with two wavefronts (64 x 128: 13.9 and 10.1 with
// 16 right-hand sides, but slower with one), nor wider ones a row a wavefront.
bool solve_vc_wg_supported(const GeomVC &g, int s)
{
    auto whole = [s](int tiles, int overlap) { return tiles == 1 || overlap >= 2 * ((int64_t)s - 1); };
    return g.reg && g.nx <= 64 && g.ny <= 64 && whole(g.ntx, g.ox) && whole(g.nty, g.oy);
}

hipError_t launch_solve_vc_wg(const GeomVC &g, int64_t batch, int64_t stride, int s, const double *f, double *u,
                              int64_t c_begin, int64_t c_end, int64_t maxc, double tol, bool every, Ctrl *ctrls,
                              hipStream_t st)
{
    if (!solve_vc_wg_supported(g, s) || batch < 1 || batch > 1 << 22 || c_begin < 0 || c_end <= c_begin ||
        c_end - 1 > maxc || s < 1)
        return hipErrorInvalidValue;
    auto at = [&](auto launch) {
        return launch(g, batch, stride, s, f, u, c_begin, c_end, maxc, tol, every, ctrls, st);
    };
    // rows a wavefront: the fewest that hold the grid in eight
    if (g.ny <= 16) return at(launch_vc_wg<2>);
    if (g.ny <= 24) return at(launch_vc_wg<3>);
    if (g.ny <= 32) return at(launch_vc_wg<4>);
    if (g.ny <= 48) return at(launch_vc_wg<6>);
    return at(launch_vc_wg<8>);
}

}  // namespace hj
