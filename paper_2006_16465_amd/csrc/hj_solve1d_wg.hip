// hj_solve1d_wg.hip -- a whole 1D hierarchical solve inside one workgroup.
//
// When every tile of a 1D problem fits in one workgroup (at most 16 register
// tiles, one per wavefront) and the grid fits in LDS, a cycle needs no kernel
// launch of its own.  The two global iterates sit in LDS and f in registers;
// each wavefront runs its tile's cycle in registers (load with a frozen halo,
// s sweeps, write-back of the owned points: Sec. 3.3, with the overlap of
// Sec. 3.5; the update of reg_sweep_1d); the workgroup barrier that ends the
// cycle is the global synchronisation between cycles.  The residual of the
// iterate a cycle reads is reduced in the same pass and judged during the
// next cycle, before that one's write-back, so the solve stops at the same
// iterate as the per-cycle path, and the iterates agree with it bit for bit.
#include <algorithm>

#include "hj_launch.h"
#include "hj_tiles.h"
#include "hj_wg.h"

namespace hj {
namespace {

constexpr int kWgThreads = 1024;              // launch bound; a launch has one wavefront per tile
constexpr int kWgMaxTiles = kWgThreads / 64;  // 16
constexpr size_t kWgLdsCap = 150 * 1024;      // three arrays of the grid's size, at most
constexpr size_t kWgLdsDefault = 60 * 1024;   // without the device's opt-in limit

// Most bytes of three arrays of the grid's size (f and the two iterates; f has
// moved to registers, the limit stays what callers know) on the current device: the
// opt-in limit per workgroup (160 KiB on gfx950) less the static arrays,
// capped at kWgLdsCap; 60 KiB if the device does not report it.
size_t wg_max_lds()
{
    static size_t cache[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return kWgLdsDefault;
    if (!cache[dev]) {
        int v = 0;
        size_t lim = kWgLdsDefault;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeSharedMemPerBlockOptin, dev) == hipSuccess &&
            v > 2048)
            lim = std::min(kWgLdsCap, std::max(kWgLdsDefault, (size_t)v - 1024));
        cache[dev] = lim;
    }
    return cache[dev];
}

// LDS of a solve: two iterates, each between its two boundary zeros.
size_t wg_lds(int64_t n, size_t es) { return 2 * (size_t)(n + 2) * es; }

// Cycles [c_begin, c_end) of one solve by the calling workgroup (one
// wavefront per tile); c_end <= maxc + 1.  The pass for c == maxc runs no
// sweep (it only evaluates the residual of iterate maxc).  x holds iterate
// c_begin on entry and, on return, the iterate the solve stopped at
// (tolerance mode) or iterate c_end (c_end <= maxc) / maxc.  EVERY: judge
// every iterate (tolerance mode), else only iterates 0 and maxc.  A solve
// that has stopped returns at once.  MASK: the grid is shorter than its one
// tile.  SL: slots of the residual tree (8 or 16, at least the tiles).
//
// What bounds it: the serial chain of a cycle (few wavefronts, nothing to
// hide a latency with), and VALU issue where many copies share a compute
// unit.  So f, its scaled form and the lane's part in the residual stay in
// registers for the whole solve; the two iterates in LDS have a zero on either
// side, so every load is unconditional and the neighbours of a lane's run
// come with it (the first sweep needs no DPP); lanes 0 and 63 keep the frozen
// halo in the DPP destination itself; the cross-lane steps of the residual
// sum lie between the sweeps; and the verdict on iterate c is formed during
// cycle c + 1, from sums read at its start, just before that cycle's
// write-back (which would overwrite iterate c).  Measured against the generic
// tile body run in a loop, judged in line: N = 256 (64-point tiles, s = 8,
// overlap 14) 0.97 -> 0.58 us a cycle, N = 5000 (512-point tiles, s = 24,
// overlap 46) 5.29 -> 3.96 us, 1024 copies of N = 1024 (256-point tiles,
// s = 32, overlap 62) 7.1 -> 5.7 us a cycle of them all, of which VALU issue
// takes about 4.3.
template <typename T, int TT, bool MASK, int SL, bool EVERY>
__device__ __forceinline__ void solve_body(const Geom1 &g, const T *__restrict__ f, T *__restrict__ x, int s,
                                           int64_t c_begin, int64_t c_end, int64_t maxc, double tol,
                                           Ctrl *ctrl, T *smem, double (&red)[2][kWgMaxTiles])
{
    constexpr int P = TT / 64;
    // Solve state, identical in every thread (read before any thread of this
    // launch writes the block: the writes below follow at least one barrier).
    WgJudge J;
    J.status = ctrl->status;
    if (EVERY && J.status != ST_RUNNING) return;
    J.r0sq = ctrl->r0sq;
    J.last = ctrl->last_rsq;
    J.done = ctrl->done_cycle;
    J.tol = tol;
    J.set_lim();

    const int n = (int)g.n;
    const int nth = (int)blockDim.x;
    const int pitch = n + 2;  // an iterate between its two boundary zeros
    T *b0 = smem + 1;
    for (int i = (int)threadIdx.x; i < n; i += nth) b0[i] = x[i];
    if (threadIdx.x < 4) smem[(threadIdx.x >> 1) * pitch + (threadIdx.x & 1) * (n + 1)] = T(0);
    if (threadIdx.x < 2 * kWgMaxTiles) red[threadIdx.x / kWgMaxTiles][threadIdx.x % kWgMaxTiles] = 0.0;

    const int lane = (int)threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const bool live = wave < (int)g.nt;
    const int tile = live ? wave : 0;
    const int x0 = axis_origin(n, TT, g.o, tile);
    const int l0 = lane * P;
    const int lo = live ? axis_own_begin(n, TT, g.o, tile) - x0 - l0 : 0;
    const int hi = live ? axis_own_end(n, TT, g.o, tile, (int)g.nt) - x0 - l0 : 0;
    // LDS place of the lane's point i relative to the iterate (points past a
    // short grid read its right zero)
    auto at = [&](int i) { return MASK ? min(l0 + i, n) : x0 + l0 + i; };
    T fv[P], fh[P];
    double own[P];  // 1 where the tile owns the point, else 0
#pragma unroll
    for (int i = 0; i < P; ++i) {
        fv[i] = live && (!MASK || l0 + i < n) ? f[x0 + l0 + i] : T(0);
        fh[i] = (T(g.hh) * fv[i]) * T(0.5);
        own[i] = i >= lo && i < hi ? 1.0 : 0.0;
    }
    __syncthreads();

    T a[P], b[P], lft, rgt;
    auto load = [&](const T *xin) {
#pragma unroll
        for (int i = 0; i < P; ++i) a[i] = xin[at(i)];
        lft = xin[at(0) - 1];
        rgt = xin[at(P)];
    };
    // the lane's share of ||r||^2 over the owned points, from the values just
    // loaded (own * rr is 0 elsewhere; a point that is not finite is some
    // tile's own, so the total is not finite either way)
    auto residual = [&]() {
        double acc = 0.0;
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const double w = (double)(i > 0 ? a[i - 1] : lft);
            const double e = (double)(i + 1 < P ? a[i + 1] : rgt);
            const double rr = (double)fv[i] - g.w1 * (__builtin_fma(2.0, (double)a[i], -w) - e);
            acc = __builtin_fma(own[i] * rr, rr, acc);
        }
        return acc;
    };
    // u -> v, its outer neighbours in lft and rgt
    auto update = [&](const T(&u)[P], T(&v)[P]) {
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const T w = i > 0 ? u[i - 1] : lft;
            const T e = i + 1 < P ? u[i + 1] : rgt;
            const T r = __builtin_fma(w + e, T(0.5), fh[i]);
            v[i] = MASK ? (l0 + i < n ? r : T(0)) : r;
        }
    };
    auto sweep = [&](const T(&u)[P], T(&v)[P]) {
        lft = dpp_move<kDppWaveShr1>(lft, u[P - 1]);
        rgt = dpp_move<kDppWaveShl1>(rgt, u[0]);
        update(u, v);
    };
    auto post = [&](int par, double sum) {
        if (lane == 63) red[par][wave] = sum;
    };
    int64_t c = c_begin;
    const int64_t c_sweep = c_end < maxc ? c_end : maxc;  // cycles with sweeps: [c_begin, c_sweep)
    int par = 0;        // buffer and slots of iterate c
    bool stop = false;  // the solve stopped at iterate c - 1 (its buffer is the other one)
    for (; c < c_sweep; ++c) {
        const T *xin = b0 + par * pitch;
        T *xout = b0 + (par ^ 1) * pitch;
        double tot = tree_sum<SL>(red[par ^ 1]);  // of iterate c - 1 (before the first: unused)
        if (live) {
            load(xin);
            double mine = residual();
            update(a, b);
            int k = 1;
            if (s >= 8) {
                sweep(b, a);
                mine = wave_step<0>(mine);
                sweep(a, b);
                mine = wave_step<1>(mine);
                sweep(b, a);
                mine = wave_step<2>(mine);
                sweep(a, b);
                mine = wave_step<3>(mine);
                asm volatile("" : "+v"(tot));  // keeps the tree here, between the sweeps
                sweep(b, a);
                mine = wave_step<4>(mine);
                sweep(a, b);
                mine = wave_step<5>(mine);
                k = 7;
            } else {
                mine = wave_sum63(mine);
            }
            for (; k + 1 < s; k += 2) {
                sweep(b, a);
                sweep(a, b);
            }
            post(par, mine);
            if (k < s) {
                sweep(b, a);
#pragma unroll
                for (int i = 0; i < P; ++i) b[i] = a[i];
            }
        }
        // the verdict on iterate c - 1, before its buffer is overwritten
        if (EVERY && J.far(tot)) {
            J.last = tot;
        } else if (c > c_begin && (EVERY || c == 1)) {
            J.take(c - 1, tot);
            if (EVERY && J.status != ST_RUNNING) {
                stop = true;
                break;
            }
        }
        if (live) {
#pragma unroll
            for (int i = 0; i < P; ++i)
                if (own[i] != 0.0) xout[x0 + l0 + i] = b[i];
        }
        // The one barrier of a cycle: its write-back and wavefront sums are
        // visible after it, and every read of xin and of the other slots is
        // done before the next cycle overwrites them.
        __syncthreads();
        par ^= 1;
    }
    if (!stop && c > c_begin && (EVERY || c == 1)) {
        J.take(c - 1, tree_sum<SL>(red[par ^ 1]));
        stop = EVERY && J.status != ST_RUNNING;
    }
    int buf = stop ? par ^ 1 : par;
    int64_t k_end = stop ? c - 1 : c;
    if (!stop && c_end == maxc + 1) {
        // the residual of iterate maxc
        if (live) {
            load(b0 + par * pitch);
            post(par, wave_sum63(residual()));
        }
        __syncthreads();
        J.take(maxc, tree_sum<SL>(red[par]));
        k_end = EVERY && J.status != ST_RUNNING ? maxc : c_end;
    }
    for (int i = (int)threadIdx.x; i < n; i += nth) x[i] = b0[buf * pitch + i];
    if (threadIdx.x == 0) {
        ctrl->r0sq = J.r0sq;
        ctrl->last_rsq = J.last;
        ctrl->iter = k_end;
        ctrl->done_cycle = J.done;
        ctrl->status = J.status;
    }
}

// The body for a grid of one short tile (whose other slots stay 0, whatever
// the workgroup was launched for) or of whole tiles (uniform).
template <typename T, int TT, int SL>
__device__ __forceinline__ void solve_any(const Geom1 &g, const T *__restrict__ f, T *__restrict__ x, int s,
                                          int64_t c_begin, int64_t c_end, int64_t maxc, double tol, int every,
                                          Ctrl *ctrl, T *smem, double (&red)[2][kWgMaxTiles])
{
    auto go = [&]<bool MASK, int S, bool EVERY>() {
        solve_body<T, TT, MASK, S, EVERY>(g, f, x, s, c_begin, c_end, maxc, tol, ctrl, smem, red);
    };
    if (every) {
        if (g.n < TT) go.template operator()<true, 8, true>();
        else go.template operator()<false, SL, true>();
    } else {
        if (g.n < TT) go.template operator()<true, 8, false>();
        else go.template operator()<false, SL, false>();
    }
}

// One solve; launched with 64 g.nt threads.
template <typename T, int TT, int SL>
__global__ __launch_bounds__(64 * SL) void k_solve1d_wg(Geom1 g, const T *__restrict__ f, T *__restrict__ x,
                                                        int s, int64_t c_begin, int64_t c_end, int64_t maxc,
                                                        double tol, int every, Ctrl *ctrl)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[2][kWgMaxTiles];  // wavefront sums, by cycle parity
    solve_any<T, TT, SL>(g, f, x, s, c_begin, c_end, maxc, tol, every, ctrl, (T *)smem, red);
}

// Workgroup b solves problem b of a batch; launched with 64 max(nt) threads.
template <typename T, int TT, int SL>
__global__ __launch_bounds__(64 * SL) void k_solve1d_wg_batch(const WgProb *__restrict__ probs, int s,
                                                              int64_t c_begin, int64_t c_end, int64_t maxc,
                                                              double tol, int every, Ctrl *ctrls)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[2][kWgMaxTiles];
    const WgProb q = probs[blockIdx.x];
    solve_any<T, TT, SL>(q.g, (const T *)q.f, (T *)q.x, s, c_begin, c_end, maxc, tol, every, ctrls + blockIdx.x,
                         (T *)smem, red);
}

__global__ void k_ctrl_init_n(Ctrl *ctrls, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    Ctrl c;
    c.r0sq = 0.0;
    c.last_rsq = 0.0;
    c.iter = 0;
    c.done_cycle = -1;
    c.stop_at = INT64_MAX;
    c.status = ST_RUNNING;
    c.pad = 0;
    c.sw_tol = -1.0;
    c.sw_min_c = 0;
    c.host = nullptr;
    ctrls[i] = c;
}

template <typename T>
hipError_t launch_t(const Geom1 &g, int s, const void *f, void *x, int64_t c_begin, int64_t c_end, int64_t maxc,
                    double tol, bool every, Ctrl *ctrl, hipStream_t st)
{
    const size_t lds = wg_lds(g.n, sizeof(T));
    const int ev = every ? 1 : 0;
    const unsigned nth = 64u * (unsigned)g.nt;  // one wavefront per tile
    auto go = [&](auto kernel) -> hipError_t {
        if (hipError_t e = allow_lds(kernel, lds); e != hipSuccess) return e;
        kernel<<<1, nth, lds, st>>>(g, (const T *)f, (T *)x, s, c_begin, c_end, maxc, tol, ev, ctrl);
        return hipGetLastError();
    };
    switch (g.t) {
    case 64: return g.nt <= 8 ? go(k_solve1d_wg<T, 64, 8>) : go(k_solve1d_wg<T, 64, 16>);
    case 128: return g.nt <= 8 ? go(k_solve1d_wg<T, 128, 8>) : go(k_solve1d_wg<T, 128, 16>);
    case 256: return g.nt <= 8 ? go(k_solve1d_wg<T, 256, 8>) : go(k_solve1d_wg<T, 256, 16>);
    case 512: return g.nt <= 8 ? go(k_solve1d_wg<T, 512, 8>) : go(k_solve1d_wg<T, 512, 16>);
    default: return hipErrorInvalidValue;
    }
}

template <typename T>
hipError_t launch_batch_t(int tt, const WgProb *probs, int64_t nprob, int64_t max_n, int64_t max_nt, int s,
                          int64_t c_begin, int64_t c_end, int64_t maxc, double tol, bool every, Ctrl *ctrls,
                          hipStream_t st)
{
    const size_t lds = wg_lds(max_n, sizeof(T));
    const int ev = every ? 1 : 0;
    const unsigned nth = 64u * (unsigned)max_nt;
    auto go = [&](auto kernel) -> hipError_t {
        if (hipError_t e = allow_lds(kernel, lds); e != hipSuccess) return e;
        return in_launches(nprob, (int)nth, [&](int64_t first, int64_t n) {
            kernel<<<(unsigned)n, nth, lds, st>>>(probs + first, s, c_begin, c_end, maxc, tol, ev, ctrls + first);
            return hipGetLastError();
        });
    };
    switch (tt) {
    case 64: return max_nt <= 8 ? go(k_solve1d_wg_batch<T, 64, 8>) : go(k_solve1d_wg_batch<T, 64, 16>);
    case 128: return max_nt <= 8 ? go(k_solve1d_wg_batch<T, 128, 8>) : go(k_solve1d_wg_batch<T, 128, 16>);
    case 256: return max_nt <= 8 ? go(k_solve1d_wg_batch<T, 256, 8>) : go(k_solve1d_wg_batch<T, 256, 16>);
    case 512: return max_nt <= 8 ? go(k_solve1d_wg_batch<T, 512, 8>) : go(k_solve1d_wg_batch<T, 512, 16>);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

bool solve1d_wg_supported(const Geom1 &g, int dt)
{
    const size_t es = dt == F64 ? sizeof(double) : sizeof(float);
    const bool tile = g.t == 64 || g.t == 128 || g.t == 256 || g.t == 512;
    return tile && g.nt >= 1 && g.nt <= kWgMaxTiles && 3 * (size_t)g.n * es <= wg_max_lds();
}

hipError_t launch_solve1d_wg(int dt, const Geom1 &g, int s, const void *f, void *x, int64_t c_begin,
                             int64_t c_end, int64_t maxc, double tol, bool every, Ctrl *ctrl, hipStream_t st)
{
    if (!solve1d_wg_supported(g, dt) || c_begin < 0 || c_end <= c_begin || c_end - 1 > maxc || s < 1)
        return hipErrorInvalidValue;
    if (dt == F64) return launch_t<double>(g, s, f, x, c_begin, c_end, maxc, tol, every, ctrl, st);
    return launch_t<float>(g, s, f, x, c_begin, c_end, maxc, tol, every, ctrl, st);
}

hipError_t launch_solve1d_wg_batch(int dt, int tt, const WgProb *probs, int64_t nprob, int64_t max_n,
                                   int64_t max_nt, int s, int64_t c_begin, int64_t c_end, int64_t maxc, double tol,
                                   bool every, Ctrl *ctrls, hipStream_t st)
{
    const size_t es = dt == F64 ? sizeof(double) : sizeof(float);
    if (nprob < 1 || nprob > INT32_MAX || max_nt < 1 || max_nt > kWgMaxTiles || max_n < 1 ||
        3 * (size_t)max_n * es > wg_max_lds() || c_begin < 0 || c_end <= c_begin || c_end - 1 > maxc || s < 1)
        return hipErrorInvalidValue;
    if (dt == F64) return launch_batch_t<double>(tt, probs, nprob, max_n, max_nt, s, c_begin, c_end, maxc, tol, every, ctrls, st);
    return launch_batch_t<float>(tt, probs, nprob, max_n, max_nt, s, c_begin, c_end, maxc, tol, every, ctrls, st);
}

hipError_t launch_ctrl_init_n(Ctrl *ctrls, int64_t n, hipStream_t st)
{
    if (n < 1) return hipSuccess;
    k_ctrl_init_n<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(ctrls, n);
    return hipGetLastError();
}

}  // namespace hj
