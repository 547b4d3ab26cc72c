// hj_vc.hip -- variable-coefficient diffusion -div(a grad u) = f on the 2D
// grid: the hierarchical cycle, the residual, and the gradient of a loss with
// respect to the node coefficients a (adjoint face products).
//
// The operator, its face weights and the cycle body live in hj_vc_tile.h.
#include <hip/hip_runtime.h>

#include <algorithm>

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

// Rows a wavefront: the fewest that hold the grid in eight wavefronts.
static int vc_wg_rows(int ny) { return ny <= 16 ? 2 : ny <= 24 ? 3 : ny <= 32 ? 4 : ny <= 48 ? 6 : 8; }

// Grids of at most 64 x 64 points whose cycle is s sweeps of the whole grid.
// Higher ones do not fit a SIMD's registers with two wavefronts (64 x 128:
// 13.9 and 10.1 us a cycle of 16 right-hand sides by tiles and here, but slower
// with one), nor wider ones a row a wavefront.
bool solve_vc_wg_supported(const GeomVC &g, int s)
{
    auto whole = [s](int tiles, int overlap) { return tiles == 1 || overlap >= 2 * ((int64_t)s - 1); };
    return g.reg && g.nx <= 64 && g.ny <= 64 && whole(g.ntx, g.ox) && whole(g.nty, g.oy);
}

// Whether they run here: s sweeps must not cost more beyond the tile kernels'
// s sweeps than what those pay for a cycle's launches, loads and stores.  In us,
// for b right-hand sides:
// - a sweep here takes its chain, by the rows of a wavefront, or its issue, 24
//   ps a row and right-hand side, of 64 lanes whatever the grid's width;
// - a sweep of the tiles takes their chain, by a tile's points (the LDS body's
//   is longer), or 0.34 ps a point;
// - a cycle of the tiles takes 1 and more beside its sweeps with one right-hand
//   side, and with several (a launch to judge them) 5 and what grows with them.
// So wide grids run here (us a cycle by tiles / here, 64 x 64, s = 8: one
// right-hand side 8.8 / 3.9, 64 14.0 / 4.0, 8 192 248 / 134), narrow or low
// ones while right-hand sides or sweeps are few (3 x 64, s = 8: 512 of them
// 15.1 / 9.2, 2 048 26.7 / 35.7; 16 x 16: 2 048, s = 8 14.7 / 9.6, s = 32 20.0 /
// 29.6; 32 x 32: 2 048, s = 8 23.1 / 16.3, s = 32 40.0 / 53.6).  The numbers were
// fitted to 891 pairs of times over 26 shapes, 1 to 8 192 right-hand sides and
// s = 3 to 128; the way taken is within 5 % of the faster one in all but 13, and 27
// % from it at most (32 x 64 as one tile, one right-hand side, s = 20).
bool solve_vc_wg_faster(const GeomVC &g, int s, int64_t batch)
{
    const double b = (double)batch, pts = (double)g.tx * g.ty;
    const int rows = vc_wg_rows(g.ny), padded = (g.ny + rows - 1) / rows * rows;
    const double here = std::max(0.14 + 0.023 * rows, 2.4e-5 * b * padded);
    const double chain = (0.13 + 5.3e-5 * pts) * (vc_reg(g) ? 1.0 : 1.2);
    const double tiles = std::max(chain, 3.4e-7 * b * g.ntx * g.nty * pts);
    const double cycle = batch == 1 ? 0.91 + 7.3e-4 * pts : 4.9 + b * (1.3e-3 + 3.9e-6 * g.nx * g.ny);
    return s * (here - tiles) <= cycle;
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
    switch (vc_wg_rows(g.ny)) {
    case 2: return at(launch_vc_wg<2>);
    case 3: return at(launch_vc_wg<3>);
    case 4: return at(launch_vc_wg<4>);
    case 6: return at(launch_vc_wg<6>);
    default: return at(launch_vc_wg<8>);
    }
}

}  // namespace hj
