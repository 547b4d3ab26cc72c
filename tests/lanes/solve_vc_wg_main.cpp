// The one-workgroup variable-coefficient solve (hj_solve_vc_wg.h) run as
// lanes on the CPU: for every order of its wavefronts it must give the
// iterate, the verdict and the norms of whole-grid sweeps written out here.
#include <hip/hip_runtime.h>

#include <cstring>
#include <random>

#include "hj_solve_vc_wg.h"

namespace {

struct Problem {
    hj::GeomVC g;
    std::vector<double> a, f, u0;
};

// arguments of the run in hand
hj::GeomVC G;
const double *F;
double *U;
int S, EVERY;
int64_t MAXC;
double TOL;
hj::Ctrl *C;

template <int R, bool MASK>
void kernel()
{
    hj::k_solve_vc_wg<R, MASK>(G, F, U, 0, S, 0, MAXC + 1, MAXC, TOL, EVERY, C);
}

// value at (r, q) of an iterate, 0 beyond the grid
struct Ref {
    const Problem &p;
    double at(const std::vector<double> &x, int r, int q) const
    {
        return r >= 0 && r < p.g.ny && q >= 0 && q < p.g.nx ? x[(size_t)r * p.g.ld + q] : 0.0;
    }
    // one sweep of x, or its squared residual norm
    double pass(const std::vector<double> &x, std::vector<double> *to) const
    {
        const hj::GeomVC &g = p.g;
        double sum = 0.0;
        for (int r = 0; r < g.ny; ++r)
            for (int q = 0; q < g.nx; ++q) {
                const double *n = p.a.data() + (size_t)(r + 1) * g.lda + q + 1;
                const double w = 0.5 * (n[0] + n[-1]) * g.ihx2, e = 0.5 * (n[0] + n[1]) * g.ihx2;
                const double s = 0.5 * (n[0] + n[-g.lda]) * g.ihy2, t = 0.5 * (n[0] + n[g.lda]) * g.ihy2;
                const double c = at(x, r, q), uw = at(x, r, q - 1), ue = at(x, r, q + 1);
                const double us = at(x, r - 1, q), ut = at(x, r + 1, q), f = p.f[(size_t)r * g.ld + q];
                if (to) {
                    (*to)[(size_t)r * g.ld + q] =
                        (f + ((w * uw + e * ue) + (s * us + t * ut))) * (1.0 / ((w + e) + (s + t)));
                } else {
                    const double rr = f - ((w * (c - uw) + e * (c - ue)) + (s * (c - us) + t * (c - ut)));
                    sum += rr * rr;
                }
            }
        return sum;
    }
};

int failures = 0;

template <int R, bool MASK>
void check(int nx, int ny)
{
    Problem p;
    const int ld = nx + 1, lda = nx + 3;
    std::mt19937 gen((unsigned)(nx * 100 + ny));
    std::normal_distribution<double> normal;
    p.g = hj::GeomVC{};
    p.g.nx = nx;
    p.g.ny = ny;
    p.g.ld = ld;
    p.g.lda = lda;
    p.g.ihx2 = (nx + 1.0) * (nx + 1.0);
    p.g.ihy2 = 0.7 * p.g.ihx2;
    for (int i = 0; i < (ny + 2) * lda; ++i) p.a.push_back(std::exp(0.5 * normal(gen)));
    for (int i = 0; i < ny * ld; ++i) p.f.push_back(1e3 * normal(gen)), p.u0.push_back(normal(gen));
    p.g.a = p.a.data();
    const Ref ref{p};
    const int nw = (ny + R - 1) / R;
    std::vector<std::vector<int>> orders;
    for (int last = 0; last < nw; ++last) {  // every wavefront after all others once
        std::vector<int> o;
        for (int w = 0; w < nw; ++w)
            if (w != last) o.push_back(w);
        o.push_back(last);
        orders.push_back(o);
    }
    for (int s : {1, 2, 3, 4})
        for (int maxc : {1, 2}) {
            std::vector<std::vector<double>> x{p.u0};
            std::vector<double> rsq{ref.pass(p.u0, nullptr)};
            for (int c = 0; c < maxc; ++c) {
                std::vector<double> y = x.back(), z = y;
                for (int k = 0; k < s; ++k) {
                    ref.pass(y, &z);
                    y.swap(z);
                }
                x.push_back(y);
                rsq.push_back(ref.pass(y, nullptr));
            }
            // no tolerance, one never met, and one met at each iterate in turn
            std::vector<double> tols{-1.0, 1e-100};
            for (int c = 1; c <= maxc; ++c) tols.push_back(std::sqrt(rsq[c] / rsq[0]) * (1 + 1e-9));
            for (double tol : tols)
                for (int every : tol > 0.0 ? std::vector<int>{1} : std::vector<int>{0, 1}) {
                    int stop = maxc;
                    bool met = false;
                    for (int c = 0; c <= maxc && !met; ++c)
                        if (tol > 0.0 && std::sqrt(rsq[c] / rsq[0]) <= tol) stop = c, met = true;
                    for (const std::vector<int> &order : orders) {
                        std::vector<double> u = p.u0;
                        hj::Ctrl ctrl{};
                        ctrl.done_cycle = -1;
                        G = p.g, F = p.f.data(), U = u.data(), S = s, EVERY = every, MAXC = maxc, TOL = tol, C = &ctrl;
                        lanes::run(kernel<R, MASK>, nw, order);
                        const bool same = std::memcmp(u.data(), x[stop].data(), u.size() * 8) == 0;
                        // sums of at most 4096 squares in another order: 4096 x 2^-53 of each
                        auto near = [](double got, double want) { return std::fabs(got - want) <= 1e-12 * want; };
                        const bool verdict = (ctrl.status == hj::ST_CONVERGED) == met &&
                                             (!met || ctrl.done_cycle == stop);
                        if (!same || !verdict || !near(ctrl.r0sq, rsq[0]) || !near(ctrl.last_rsq, rsq[stop])) {
                            ++failures;
                            std::printf("%d x %d s=%d max_cycles=%d tol=%g every=%d, wavefront %d first, %d last: iterate %s, "
                                        "status %d at %d, r0 %.17g (%.17g), last %.17g (%.17g)\n",
                                        nx, ny, s, maxc, tol, every, order.front(), order.back(), same ? "right" : "WRONG",
                                        (int)ctrl.status, (int)ctrl.done_cycle, ctrl.r0sq, rsq[0], ctrl.last_rsq, rsq[stop]);
                        }
                    }
                }
        }
}

}  // namespace

int main()
{
    check<2, true>(9, 2);    // one wavefront
    check<2, true>(64, 5);   // its last wavefront holds one row
    check<3, true>(5, 9);
    check<2, false>(64, 6);  // whole rows and wavefronts
    check<8, true>(33, 20);
    std::printf("%d failures\n", failures);
    return failures != 0;
}
