// hj_device.h -- device-side building blocks shared by the HIP kernels:
// the control block of a solve, the tile partition, the XCD-aware block
// mapping and the deterministic FP64 residual reduction.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hj {

// Device-resident state of one solve.  Cycle kernels reduce the residual of
// the iterate they read and judge it on the device (see Red below), so the
// host only polls this block now and then.
struct Ctrl {
    double r0sq;         // ||r_0||^2
    double last_rsq;     // ||r_c||^2 of the latest judged iterate
    int64_t iter;        // one past the latest judged iterate
    int64_t done_cycle;  // first c that met the tolerance (or went non-finite); -1 otherwise
    int64_t stop_at;     // cycle kernels evaluating iterate k >= stop_at return at once
    int32_t status;      // 0 running, 1 converged, 2 non-finite, 3 stopped at max_cycles, 4 switch
    int32_t pad;
    // Optional hand-over point (sw_tol < 0: none).  The first iterate c with
    // a relative residual <= sw_tol (and above the tolerance) ends the solve
    // with ST_SWITCH if c >= sw_min_c; otherwise the solve runs on to the
    // tolerance.  The decision is taken once: sw_tol is set to -1 after it.
    double sw_tol;
    int64_t sw_min_c;
    // Pinned host memory that gets the verdict when it falls (r0sq, last_rsq,
    // done_cycle, then status), or nullptr.  A host that waits for an event
    // between cycles finds it there without a copy on the stream.
    Ctrl *host;
};

enum : int32_t { ST_RUNNING = 0, ST_CONVERGED = 1, ST_NONFINITE = 2, ST_LIMIT = 3, ST_SWITCH = 4 };

// ---------------------------------------------------------------------------
// Tile partition along one axis (subdomains of Sec. 3.3, overlap of Sec. 3.5).
// n points, tile t, overlap o (0 <= o < t).  n <= t: one tile of n points.
// Otherwise tiles start every t - o points; the last starts at n - t.
// ---------------------------------------------------------------------------
__host__ __device__ inline int axis_count(int n, int t, int o)
{
    return n <= t ? 1 : (n - o + (t - o) - 1) / (t - o);
}

__host__ __device__ inline int axis_origin(int n, int t, int o, int i)
{
    if (n <= t) return 0;
    const int st = i * (t - o);
    return st > n - t ? n - t : st;
}

// First point tile i writes back: the midpoint (rounded up) of its overlap
// with tile i - 1; the left neighbour keeps the lower half.
__host__ __device__ inline int axis_own_begin(int n, int t, int o, int i)
{
    if (i == 0) return 0;
    const int ext = n < t ? n : t;
    const int a = axis_origin(n, t, o, i);
    const int shared_pts = axis_origin(n, t, o, i - 1) + ext - a;
    return a + (shared_pts + 1) / 2;
}

__host__ __device__ inline int axis_own_end(int n, int t, int o, int i, int count)
{
    return i == count - 1 ? n : axis_own_begin(n, t, o, i + 1);
}

// Division by a number known on the host: t / d for t < 2^31 by one high
// product with m = floor((2^32 - 1) / d), which is q or q - 1, and a
// correction.  (A general 32-bit division is some twenty dependent
// instructions in front of every tile's loads.)
struct FastDiv {
    unsigned d, m;
};

inline FastDiv fast_div(int64_t d)
{
    const unsigned u = d >= 1 && d <= INT32_MAX ? (unsigned)d : 1u;
    return FastDiv{u, 0xffffffffu / u};
}

__device__ __forceinline__ unsigned quot(unsigned t, const FastDiv &f)
{
    const unsigned q = __umulhi(t, f.m);
    return t - q * f.d >= f.d ? q + 1 : q;
}

// The order in which a 2D grid's tiles are walked: vertical strips of sw tile
// columns (the last one narrower), row by row inside a strip.
struct Walk {
    int ntx, sw;
    FastDiv strip;  // tiles of a whole strip
    FastDiv col;    // tile columns of a whole strip
    FastDiv last;   // tile columns of the last strip
};

// Strips of equal width whose row of tiles moves at most kStripBytes (large:
// the grid is one to be walked in strips).  An XCD works on a contiguous run of
// the walk, about 64 tiles at a time, so the overlap (or halo) rows that
// vertical neighbours share are read again while its 4 MB L2 still holds them;
// row by row over the whole grid they come back after tiles_x tiles.  Measured
// at 4096^2, us per FP64 cycle with residual, whole rows / strips: 32 x 32
// tiles 99 / 88 (3.1 MB a row; strips of 16, 24 and 43 columns alike), 64 x 32
// o = 14 126 / 117, 64 x 64 o = 22 135 / 132, 64 x 128 o = 22 144 / 142.
//
// FP64 grids are large where their tiles move more than the memory-side cache
// holds (kLargeF64), the parts that overlap counted each time: 3000^2, 32 x 32,
// s = 4, overlap 6 (330 MB of tiles, 216 MB of grid), without residual 47 / 42 us;
// 3300^2, s = 2, overlap 2 (297 MB) 58.4 / 55.8.  FP32 grids where the grid
// itself comes near it (kLargeF32): 32 x 32 tiles, without residual, s = 2,
// overlap 2 and s = 4, overlap 6, 4096^2 (201 MB) 36.1 / 39.0 and 38.8 / 42.6,
// 4200^2 41.5 / 44.5 and 48.2 / 48.9, 4400^2 (232 MB) 56.5 / 54.2 and 63.6 /
// 60.9, 4800^2, s = 2, 75.7 / 73.1; 3600^2 alike; 64-wide tiles within 1 % at
// 4096^2.  Strips are as wide for FP32 as for FP64 (tile_bytes of FP64 points):
// twice as wide they took 2 % more at 6000^2, s = 2 and 4.
constexpr double kLargeF64 = 256 << 20, kLargeF32 = 208 << 20;

inline Walk make_walk(int ntx, int nty, int64_t tile_bytes, bool large)
{
    constexpr int64_t kStripBytes = 3 << 19;
    const int64_t most = large ? kStripBytes / tile_bytes : ntx;
    const int cap = most < 1 ? 1 : most > ntx ? ntx : (int)most;
    const int strips = (ntx + cap - 1) / cap;
    const int sw = (ntx + strips - 1) / strips;
    const int rest = ntx % sw;
    return Walk{ntx, sw, fast_div((int64_t)sw * nty), fast_div(sw), fast_div(rest ? rest : sw)};
}

// Tile (row bi, column bj) of work index t.
__device__ __forceinline__ void tile_pos(const Walk &w, int t, int &bi, int &bj)
{
    const unsigned s = quot((unsigned)t, w.strip);
    const unsigned rest = (unsigned)t - s * w.strip.d;
    const int col0 = (int)s * w.sw;
    const FastDiv c = w.ntx - col0 < w.sw ? w.last : w.col;
    const unsigned row = quot(rest, c);
    bi = (int)row;
    bj = col0 + (int)(rest - row * c.d);
}

// ---------------------------------------------------------------------------
// Workgroups are handed to the 8 XCDs round-robin (block b runs on XCD b % 8).
// Give every XCD a contiguous run of tiles so neighbouring tiles, which read
// each other's edge points as halo, share that XCD's L2.
// ---------------------------------------------------------------------------
__device__ inline int xcd_tile(int b, int nb)
{
    constexpr int kXcd = 8;
    const int q = nb / kXcd, r = nb % kXcd;
    const int k = b % kXcd, local = b / kXcd;
    const int base = k < r ? k * (q + 1) : r * (q + 1) + (k - r) * q;
    return base + local;
}

// ---------------------------------------------------------------------------
// Deterministic sums: a wavefront by DPP steps, then wavefronts in index order.
// ---------------------------------------------------------------------------
// v from the lane CTRL selects, 0 in rows ROW_MASK leaves out.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_or_zero(double v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, ROW_MASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, ROW_MASK, 0xf, false);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// One of the six steps of a sum over the 64 lanes of a wavefront (all lanes
// active); after them lane 63 holds it.  Quads, half rows and rows of 16 by
// lane permutations, then rows 0+1 and 2+3 by broadcasts of lane 15 of a row
// into the next.
template <int STEP>
__device__ __forceinline__ double wave_step(double v)
{
    constexpr int ctrl[6] = {
        0xb1,   // quad_perm [1,0,3,2]
        0x4e,   // quad_perm [2,3,0,1]
        0x141,  // row_half_mirror
        0x140,  // row_mirror
        0x142,  // row_bcast:15 into rows 1 and 3
        0x143,  // row_bcast:31 into rows 2 and 3
    };
    constexpr int rows[6] = {0xf, 0xf, 0xf, 0xf, 0xa, 0xc};
    return v + dpp_or_zero<ctrl[STEP], rows[STEP]>(v);
}

// The sum over the wavefront, in lane 63 (a butterfly of lane shuffles goes
// through LDS, six dependent round trips of it).
__device__ __forceinline__ double wave_sum63(double v)
{
    v = wave_step<0>(v);
    v = wave_step<1>(v);
    v = wave_step<2>(v);
    v = wave_step<3>(v);
    v = wave_step<4>(v);
    return wave_step<5>(v);
}

// Sum over a workgroup of NT threads, in every thread.  red: NT / 64 doubles
// of LDS that no earlier use of the workgroup still reads.
template <int NT>
__device__ inline double block_sum(double v, double *red)
{
    v = wave_sum63(v);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 63) red[wid] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) t += red[w];
    return t;
}

// Decide convergence for iterate c from its squared residual norm.  Once a
// verdict stands the block is frozen, so last_rsq stays that of done_cycle.
__device__ inline void judge(Ctrl *ctrl, int64_t c, double rsq, double tol)
{
    if (ctrl->status != ST_RUNNING) return;
    if (c == 0) ctrl->r0sq = rsq;
    const double r0sq = ctrl->r0sq;
    ctrl->last_rsq = rsq;
    ctrl->iter = c + 1;
    const double rel = r0sq > 0.0 ? sqrt(rsq) / sqrt(r0sq) : 0.0;
    int32_t st = ST_RUNNING;
    if (!isfinite(rsq)) st = ST_NONFINITE;
    else if (rel <= tol) st = ST_CONVERGED;
    else if (ctrl->sw_tol >= 0.0 && rel <= ctrl->sw_tol) {
        if (c >= ctrl->sw_min_c) st = ST_SWITCH;
        else ctrl->sw_tol = -1.0;
    }
    if (st != ST_RUNNING) {
        ctrl->done_cycle = c;
        // workgroups of the judging kernel (it evaluates iterate c + 1) that
        // start after the verdict return at once, as do all later kernels
        __hip_atomic_store(&ctrl->stop_at, c + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&ctrl->status, st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (Ctrl *const h = ctrl->host) {
            h->r0sq = r0sq;
            h->last_rsq = rsq;
            h->done_cycle = c;
            __hip_atomic_store(&h->status, st, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

// Early exit of a cycle kernel that evaluates iterate k.  After a verdict on
// iterate c, iterate c + 1 is whole (the kernel that wrote it judged c - 1,
// which did not stop the solve); iterate c + 2 may be partial.
__device__ inline bool stopped(const Ctrl *ctrl, int64_t k)
{
    return k >= __hip_atomic_load(&ctrl->stop_at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline int32_t read_status(const Ctrl *ctrl)
{
    return __hip_atomic_load(&ctrl->status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Residual bookkeeping handed to every kernel that reduces ||r||^2.
// Each workgroup stores its partial sum in its slot of part_cur with a plain
// store.  The sum over the grid is formed by workgroup 0 of the NEXT kernel on
// the stream (the kernel boundary makes the partials visible), which judges
// iterate c - 1; no atomics and no cache-flushing fences inside the grid.
// That workgroup does nothing else: such a kernel launches one workgroup more
// than it has tiles (with a tile of its own to do after the verdict it ended
// last, about 1 us of every cycle on grids of a few hundred tiles).
struct Red {
    double *part_cur;         // this kernel's partials (one per tile or block)
    const double *part_prev;  // the previous kernel's partials
    Ctrl *ctrl;
    int64_t c;                // index of the iterate this kernel evaluates
    int nb_prev;              // partials of the previous kernel (0: nothing to judge)
    int first = 0;            // work index of the launch's first tile (kernels that run in several launches)
};

// Sum n partials in a fixed order and judge iterate c (one workgroup).
// Thread t adds chunks of 8 consecutive partials; U chunks are in flight per
// thread before any add, so a workgroup reads 2K partials or more in one memory
// latency.  U falls with the workgroup's size: 32 loads in flight a thread hold
// 64 VGPRs, more than an FP32 tile needs for its sweeps.
template <int NT>
__device__ inline void judge_partials(const double *part, int n, Ctrl *ctrl, int64_t c, double tol)
{
    __shared__ double red[NT / 64];
    constexpr int V = 8, U = NT >= 256 ? 1 : NT >= 128 ? 2 : 4;
    double acc = 0.0;
    for (int base = 0; base < n; base += NT * V * U) {
        double v[U][V];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i0 = base + (u * NT + (int)threadIdx.x) * V;
            if (i0 + V <= n) {
#pragma unroll
                for (int e = 0; e < V; ++e) v[u][e] = part[i0 + e];
            } else {
#pragma unroll
                for (int e = 0; e < V; ++e) v[u][e] = i0 + e < n ? part[i0 + e] : 0.0;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < V; ++e) acc += v[u][e];
    }
    const double tot = block_sum<NT>(acc, red);
    if (threadIdx.x == 0) judge(ctrl, c, tot, tol);
}

// Start of a kernel that reduces ||r||^2 and judges: false for workgroups
// with nothing (more) to do.  The others are numbered by judged_block.  LATE:
// the caller asks stopped() itself, once its loads are under way.
template <int NT, bool LATE = false>
__device__ inline bool judged_start(const Red &red, double tol)
{
    if (!LATE && stopped(red.ctrl, red.c)) return false;
    if (blockIdx.x > 0) return true;
    if (red.nb_prev > 0) judge_partials<NT>(red.part_prev, red.nb_prev, red.ctrl, red.c - 1, tol);
    return false;
}

// Number of this workgroup and how many there are; JUDGED: workgroup 0 left out.
template <bool JUDGED>
__device__ inline int judged_block()
{
    return (int)blockIdx.x - (JUDGED ? 1 : 0);
}

template <bool JUDGED>
__device__ inline int judged_blocks()
{
    return (int)gridDim.x - (JUDGED ? 1 : 0);
}

template <int NT>
__device__ inline void post_partial(double mine, double *slot)
{
    __shared__ double red[NT / 64];
    const double bs = block_sum<NT>(mine, red);
    if (threadIdx.x == 0) *slot = bs;
}

}  // namespace hj
