"""GPU parity: the HIP path (through the C ABI) against the CPU FP64 oracle on
the same seeded inputs.  FP64 iterates must agree within 1e-12 relative (the
kernels use the same update association and no FMA contraction, so they are
expected to agree bit for bit); FP32 iterates within 1e-5 relative of the FP64
oracle; cycles-to-tolerance must be equal."""
import ctypes
import sys

import numpy as np
import pytest

from paper_2006_16465_amd import hj
from paper_2006_16465_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    hj.load()
    yield


def dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a)).to(dtype=dtype, device="cuda")


def host(t):
    torch.cuda.synchronize()
    return t.double().cpu().numpy()


def rel(a, b):
    nb = np.linalg.norm(b)
    return np.linalg.norm(a - b) / (nb if nb > 0 else 1.0)


def gpu_cycles_2d(f, x0, h, tile, s, ncyc, overlap=(0, 0), dtype=torch.float64, method="hierarchical",
                  hy=None, lds_kernel=False):
    F, X = dev(f, dtype), dev(x0, dtype)
    info = hj.solve_2d(F, X, hx=h, hy=hy if hy else h, tile=tile, s=s, overlap=overlap, method=method,
                       rel_tol=0.0, max_cycles=ncyc, lds_kernel=lds_kernel)
    assert info.cycles == ncyc
    return host(X), info


def gpu_cycles_1d(f, x0, h, tile, s, ncyc, overlap=0, dtype=torch.float64, method="hierarchical",
                  launch_per_cycle=False):
    F, X = dev(f, dtype), dev(x0, dtype)
    info = hj.solve_1d(F, X, h, tile=tile, s=s, overlap=overlap, method=method, rel_tol=0.0,
                       max_cycles=ncyc, launch_per_cycle=launch_per_cycle)
    assert info.cycles == ncyc
    return host(X), info


# ------------------------------------------------------------------ 2D cycles, fixed counts

@pytest.mark.parametrize("s", [1, 4, 8, 16, 32])
def test_cycle2d_512_all_s_matches_oracle(orc, s):
    f, h = W.make("poisson2d_512", 0)
    x0 = np.zeros_like(f)
    for nc in (1, 2, 7, 64):
        say(f"cycle2d 512^2 s={s} cycles={nc}")
        got, info = gpu_cycles_2d(f, x0, h, (32, 32), s, nc)
        want = orc.hier_2d(f, x0, h, h, (32, 32), s, nc)
        assert rel(got, want) <= 1e-12
        assert np.array_equal(got, want), "FP64 iterates expected bit-identical"
        assert info.sweeps == nc * s


@pytest.mark.parametrize("shape", [(77, 100), (65, 33), (3, 5), (64, 130), (1, 40)])
@pytest.mark.parametrize("tile", [(32, 32), (64, 16), (16, 64)])
@pytest.mark.parametrize("overlap", [(0, 0), (4, 2), (10, 6)])
def test_cycle2d_ragged_and_overlap(orc, shape, tile, overlap):
    ny, nx = shape
    f = W.rhs_random(shape, nx * 31 + ny)
    x0 = W.rhs_random(shape, nx * 37 + ny)
    h = 1.0 / (max(nx, ny) + 1)
    ov = (min(overlap[0], tile[0] - 2), min(overlap[1], tile[1] - 2))
    for s, nc in ((1, 3), (3, 1), (16, 5)):
        say(f"cycle2d ragged {shape} tile={tile} ov={ov} s={s} nc={nc}")
        got, _ = gpu_cycles_2d(f, x0, h, tile, s, nc, ov)
        want = orc.hier_2d(f, x0, h, h, tile, s, nc, ov)
        assert np.array_equal(got, want)


def test_cycle2d_anisotropic_spacing(orc):
    ny, nx = 96, 130
    f = W.rhs_random((ny, nx), 5)
    x0 = W.rhs_random((ny, nx), 6)
    hx, hy = 1.0 / 131, 1.0 / 61
    for tile, s, nc in (((32, 32), 8, 4), ((64, 16), 5, 3)):
        say(f"cycle2d aniso tile={tile} s={s}")
        got, _ = gpu_cycles_2d(f, x0, hx, tile, s, nc, hy=hy)
        want = orc.hier_2d(f, x0, hx, hy, tile, s, nc)
        assert np.array_equal(got, want)


@pytest.mark.parametrize("tile", [(32, 16), (32, 32), (64, 16), (64, 32)])
@pytest.mark.parametrize("overlap", [(0, 0), (4, 4), (6, 2)])
def test_register_and_lds_kernels_match_oracle(orc, tile, overlap):
    """Full tiles of the register-resident shapes: both cycle kernels, several
    s (odd and even), a non-square grid that forces a right-aligned last tile."""
    ny, nx = 150, 200
    f = W.rhs_random((ny, nx), tile[0] + 3 * tile[1] + overlap[0])
    x0 = W.rhs_random((ny, nx), 7)
    h = 1.0 / 201
    for s, nc in ((1, 2), (2, 3), (7, 2), (16, 2)):
        say(f"reg/lds tile={tile} ov={overlap} s={s} nc={nc}")
        want = orc.hier_2d(f, x0, h, h, tile, s, nc, overlap)
        got, _ = gpu_cycles_2d(f, x0, h, tile, s, nc, overlap)
        assert np.array_equal(got, want), "register kernel"
        got_lds, _ = gpu_cycles_2d(f, x0, h, tile, s, nc, overlap, lds_kernel=True)
        assert np.array_equal(got_lds, want), "LDS kernel"


@pytest.mark.parametrize("tile", [(32, 32), (64, 32), (64, 64), (32, 64)])
def test_fp32_register_kernel_equals_fp32_lds_kernel(tile):
    """FP32 register tiles rotate rows through R + 1 slots in straight-line
    rounds of R + 1 sweeps with a remainder; the LDS kernel forms the same
    sums in the same order, so the two agree bit for bit for every s."""
    ny, nx = 150, 200
    f = W.rhs_random((ny, nx), 9)
    x0 = W.rhs_random((ny, nx), 10)
    for s, ov in ((1, (0, 0)), (2, (2, 2)), (3, (4, 4)), (5, (8, 8)), (7, (0, 0)), (9, (12, 12)), (12, (6, 6))):
        a, _ = gpu_cycles_2d(f, x0, 1.0 / 201, tile, s, 3, ov, dtype=torch.float32)
        b, _ = gpu_cycles_2d(f, x0, 1.0 / 201, tile, s, 3, ov, dtype=torch.float32, lds_kernel=True)
        assert np.array_equal(a, b), (tile, s, ov)


@pytest.mark.parametrize("tile", [(32, 64), (32, 128), (64, 64), (64, 128), (128, 16), (128, 32),
                                  (128, 64), (128, 128)])
@pytest.mark.parametrize("overlap", [(0, 0), (14, 14), (30, 6)])
def test_multiwave_register_kernel_matches_oracle(orc, tile, overlap):
    """Tiles held by several wavefronts (or 128 columns wide): ragged grids of a
    few tiles per axis, with and without overlap, FP64 bit for bit.  The
    sub-iteration counts cover the sweep loop's two-sweeps-per-trip form:
    s = 1 (no loop), 2 (the single leftover sweep only), 3 and 5 (whole
    trips only), 8 (trips and a leftover)."""
    ny, nx = 300, 270
    ov = (min(overlap[0], tile[0] - 2), min(overlap[1], tile[1] - 2))
    f = W.rhs_random((ny, nx), tile[0] * 7 + tile[1] + ov[0])
    x0 = W.rhs_random((ny, nx), 11 + ov[1])
    h = 1.0 / 301
    for s, nc in ((1, 2), (2, 2), (3, 3), (5, 2), (8, 2)):
        say(f"multiwave tile={tile} ov={ov} s={s} nc={nc}")
        got, _ = gpu_cycles_2d(f, x0, h, tile, s, nc, ov)
        assert np.array_equal(got, orc.hier_2d(f, x0, h, h, tile, s, nc, ov))


@pytest.mark.parametrize("tile", [(64, 64), (64, 128), (128, 64)])
def test_multiwave_register_kernel_aniso_fp32_and_exact_grid(orc, tile):
    # anisotropic spacing (general update), FP32 within 1e-5, and a grid of
    # exactly one tile (every halo is the Dirichlet boundary)
    ny, nx = 200, 260
    f = W.rhs_random((ny, nx), 3)
    x0 = W.rhs_random((ny, nx), 4)
    got, _ = gpu_cycles_2d(f, x0, 1.0 / 261, tile, 6, 3, (10, 10), hy=1.0 / 151)
    assert np.array_equal(got, orc.hier_2d(f, x0, 1.0 / 261, 1.0 / 151, tile, 6, 3, (10, 10)))
    g32, _ = gpu_cycles_2d(f, x0, 1.0 / 261, tile, 8, 20, (14, 14), dtype=torch.float32)
    assert rel(g32, orc.hier_2d(f, x0, 1.0 / 261, 1.0 / 261, tile, 8, 20, (14, 14))) <= 1e-5
    ty, tx = tile[1], tile[0]
    f1 = W.rhs_random((ty, tx), 5)
    got, _ = gpu_cycles_2d(f1, np.zeros_like(f1), 1.0 / (tx + 1), tile, 16, 2)
    assert np.array_equal(got, orc.hier_2d(f1, np.zeros_like(f1), 1.0 / (tx + 1), 1.0 / (tx + 1), tile, 16, 2))


def test_multiwave_solve_to_tolerance_matches_oracle(orc):
    f = W.rhs_2d_modes(512, 512, 16, 0.1, 6)
    h = 1.0 / 513
    X = dev(np.zeros_like(f))
    info = hj.solve_2d(dev(f), X, h, tile=(64, 128), s=8, overlap=(14, 14), rel_tol=1e-6)
    xo, co, relo, _ = orc.solve_2d(f, np.zeros_like(f), h, h, tile=(64, 128), s=8, overlap=(14, 14),
                                   tol=1e-6)
    say(f"multiwave solve 512^2: gpu cycles {info.cycles}, oracle {co}")
    assert info.cycles == co
    assert np.array_equal(host(X), xo)
    assert abs(info.rel_residual - relo) <= 1e-12 * relo


def test_128_tiles_need_full_grid():
    f = np.zeros((100, 300))
    with pytest.raises(hj.HJError):
        gpu_cycles_2d(f, f, 0.01, (64, 128), 4, 1)
    with pytest.raises(hj.HJError):
        gpu_cycles_2d(np.zeros((300, 300)), np.zeros((300, 300)), 0.01, (128, 128), 4, 1, lds_kernel=True)


@pytest.mark.parametrize("tile", [(32, 32), (64, 32)])
def test_register_kernel_solve_and_fp32(orc, tile):
    f = W.rhs_2d_modes(256, 256, 16, 0.1, 4)
    h = 1.0 / 257
    x0 = np.zeros_like(f)
    X = dev(x0)
    info = hj.solve_2d(dev(f), X, h, tile=tile, s=8, rel_tol=1e-6)
    xo, co, relo, _ = orc.solve_2d(f, x0, h, h, tile=tile, s=8, tol=1e-6)
    assert info.cycles == co
    assert np.array_equal(host(X), xo)
    assert abs(info.rel_residual - relo) <= 1e-12 * relo
    got, _ = gpu_cycles_2d(f, x0, h, tile, 16, 40, dtype=torch.float32)
    assert rel(got, orc.hier_2d(f, x0, h, h, tile, 16, 40)) <= 1e-5
    aniso, _ = gpu_cycles_2d(f, x0, h, tile, 5, 3, hy=1.0 / 129)
    assert np.array_equal(aniso, orc.hier_2d(f, x0, h, 1.0 / 129, tile, 5, 3))


@pytest.mark.parametrize("shape", [(512, 512), (77, 100), (1, 1), (200, 3)])
def test_global_sweep_2d_matches_oracle(orc, shape):
    f = W.rhs_random(shape, 41)
    x0 = W.rhs_random(shape, 42)
    h = 1.0 / (max(shape) + 1)
    for nc in (1, 7, 64):
        say(f"sweep2d {shape} sweeps={nc}")
        got, info = gpu_cycles_2d(f, x0, h, (32, 32), 1, nc, method="global")
        assert np.array_equal(got, orc.jacobi_2d(f, x0, h, h, nc))
        assert info.sweeps == nc


# ------------------------------------------------------------------ 1D

@pytest.mark.parametrize("n", [256, 1000, 37, 5, 3000])
@pytest.mark.parametrize("tile", [32, 64, 128, 256, 512, 1024])
@pytest.mark.parametrize("overlap", [0, 4, 10])
def test_cycle1d_matches_oracle(orc, n, tile, overlap):
    """Tiles of 64 points and more run register-resident (one wavefront per
    tile), 32-point tiles through LDS; both must equal the oracle bit for bit,
    also on grids shorter than one tile."""
    f = W.rhs_random(n, n + tile)
    x0 = W.rhs_random(n, n + tile + 1)
    h = 1.0 / (n + 1)
    for s, nc in ((1, 4), (16, 3), (5, 9)):
        say(f"cycle1d n={n} tile={tile} ov={overlap} s={s} nc={nc}")
        got, _ = gpu_cycles_1d(f, x0, h, tile, s, nc, overlap)
        assert np.array_equal(got, orc.hier_1d(f, x0, h, tile, s, nc, overlap))


@pytest.mark.parametrize("n", [256, 1, 2, 1025, 6144, 100000])
@pytest.mark.parametrize("per_sweep", [False, True])
def test_global_sweep_1d_matches_oracle(orc, n, per_sweep):
    """Classical sweeps: launch-free in one workgroup where the grid fits
    (n <= 6144 here), one launch per sweep otherwise or on request."""
    f = W.rhs_random(n, 3)
    x0 = W.rhs_random(n, 4)
    h = 1.0 / (n + 1)
    for nc in (1, 10):
        got, _ = gpu_cycles_1d(f, x0, h, 32, 1, nc, method="global", launch_per_cycle=per_sweep)
        assert np.array_equal(got, orc.jacobi_1d(f, x0, h, nc))


# ------------------------------------------------------------------ residual

@pytest.mark.parametrize("shape", [(512, 512), (33, 70), (1, 1)])
def test_residual_2d_matches_oracle(orc, shape):
    f = W.rhs_random(shape, 51)
    x = W.rhs_random(shape, 52)
    hx, hy = 1.0 / (shape[1] + 1), 1.0 / (shape[0] + 1)
    F, X = dev(f), dev(x)
    R = torch.empty_like(F)
    nrm = hj.residual(F, X, hx=hx, hy=hy, r_out=R)
    r, nw = orc.residual_2d(f, x, hx, hy)
    assert abs(nrm - nw) <= 1e-12 * nw
    assert np.max(np.abs(host(R) - r)) <= 1e-12 * np.max(np.abs(r))


def test_residual_1d_matches_oracle(orc):
    n = 10007
    f, x = W.rhs_random(n, 61), W.rhs_random(n, 62)
    h = 1.0 / (n + 1)
    F, X = dev(f), dev(x)
    R = torch.empty_like(F)
    nrm = hj.residual(F, X, h, r_out=R)
    r, nw = orc.residual_1d(f, x, h)
    assert abs(nrm - nw) <= 1e-12 * nw
    assert np.max(np.abs(host(R) - r)) <= 1e-12 * np.max(np.abs(r))


# ------------------------------------------------------------------ solve to tolerance

@pytest.mark.parametrize("seed", range(5))
def test_solve_1d_cycles_to_tol_match_oracle(orc, seed):
    f, h = W.make("poisson1d_n256", seed)
    x0 = np.zeros_like(f)
    for method, om, lpc in (("hierarchical", orc.HIERARCHICAL, False), ("global", orc.CLASSICAL, False),
                            ("global", orc.CLASSICAL, True)):
        say(f"solve1d n=256 seed={seed} {method} launch_per_sweep={lpc}")
        X = dev(x0)
        info = hj.solve_1d(dev(f), X, h, tile=32, s=16, method=method, rel_tol=1e-6, launch_per_cycle=lpc)
        xo, co, relo, r0o = orc.solve_1d(f, x0, h, method=om, tile=32, s=16, tol=1e-6)
        assert info.cycles == co
        assert np.array_equal(host(X), xo)
        assert abs(info.rel_residual - relo) <= 1e-12 * relo
        assert abs(info.r0_norm - r0o) <= 1e-12 * r0o


@pytest.mark.parametrize("n,tile,s,ov", [(256, 64, 8, 14), (5000, 512, 24, 46), (70000, 1024, 24, 46)])
def test_solve_1d_overlapped_register_tiles_to_tol_match_oracle(orc, n, tile, s, ov):
    """Exact-regime overlap (o = 2s - 2) with register-resident tiles, solved
    to 1e-6 from x0 = 0: same cycle count and iterate as the oracle."""
    f = W.rhs_1d_modes(n, 8, 11)
    h = 1.0 / (n + 1)
    x0 = np.zeros_like(f)
    X = dev(x0)
    say(f"solve1d n={n} tile={tile} s={s} ov={ov}")
    info = hj.solve_1d(dev(f), X, h, tile=tile, s=s, overlap=ov, rel_tol=1e-6)
    xo, co, relo, _ = orc.solve_1d(f, x0, h, tile=tile, s=s, tol=1e-6, overlap=ov)
    assert info.cycles == co > 0
    assert np.array_equal(host(X), xo)
    assert abs(info.rel_residual - relo) <= 1e-12 * relo


@pytest.mark.parametrize("s,tile,ov", [(8, (32, 32), (0, 0)), (16, (32, 32), (0, 0)), (4, (16, 16), (2, 2))])
def test_solve_2d_cycles_to_tol_match_oracle(orc, s, tile, ov):
    f = W.rhs_2d_modes(128, 128, 16, 0.1, 3)
    h = 1.0 / 129
    x0 = np.zeros_like(f)
    X = dev(x0)
    say(f"solve2d 128^2 s={s} tile={tile} ov={ov}")
    info = hj.solve_2d(dev(f), X, h, tile=tile, s=s, overlap=ov, rel_tol=1e-6, check_every=7)
    xo, co, relo, _ = orc.solve_2d(f, x0, h, h, tile=tile, s=s, tol=1e-6, overlap=ov)
    assert info.cycles == co > 0
    assert np.array_equal(host(X), xo)
    assert abs(info.rel_residual - relo) <= 1e-12 * relo


def test_solve_2d_global_cycles_to_tol_match_oracle(orc):
    f = W.rhs_2d_modes(96, 96, 8, 0.0, 1)
    h = 1.0 / 97
    x0 = np.zeros_like(f)
    X = dev(x0)
    info = hj.solve_2d(dev(f), X, h, method="global", rel_tol=1e-6)
    xo, co, _, _ = orc.solve_2d(f, x0, h, h, method=orc.CLASSICAL, tol=1e-6)
    assert info.cycles == co > 0
    assert np.array_equal(host(X), xo)


# ------------------------------------------------------------------ full size 4096^2

def test_4096_fixed_cycles_and_determinism(orc):
    f, h = W.make("poisson2d_4096", 2)
    x0 = np.zeros_like(f)
    say("4096^2 fixed 2 cycles T=32 s=16")
    got, _ = gpu_cycles_2d(f, x0, h, (32, 32), 16, 2)
    want = orc.hier_2d(f, x0, h, h, (32, 32), 16, 2)
    assert np.array_equal(got, want)
    got2, _ = gpu_cycles_2d(f, x0, h, (32, 32), 16, 2)
    assert np.array_equal(got, got2)


def test_4096_time_to_tolerance_workload_matches_oracle(orc):
    """The timed workload: 4096^2, 8 separable modes, T=32, s=16, to 1e-6."""
    f, h = W.make("poisson2d_4096", 2)
    x0 = np.zeros_like(f)
    X = dev(x0)
    say("4096^2 solve to 1e-6 (GPU)")
    info = hj.solve_2d(dev(f), X, h, tile=(32, 32), s=16, rel_tol=1e-6)
    say(f"  gpu cycles={info.cycles}; oracle solve ...")
    xo, co, relo, _ = orc.solve_2d(f, x0, h, h, tile=(32, 32), s=16, tol=1e-6, max_cycles=5000)
    assert info.cycles == co
    assert np.array_equal(host(X), xo)
    assert abs(info.rel_residual - relo) <= 1e-12 * relo
    say("4096^2 global solve to 1e-6, seed 0")
    f0, _ = W.make("poisson2d_4096", 0)
    X0 = dev(x0)
    info0 = hj.solve_2d(dev(f0), X0, h, method="global", rel_tol=1e-6)
    xo0, co0, _, _ = orc.solve_2d(f0, x0, h, h, method=orc.CLASSICAL, tol=1e-6, max_cycles=5000)
    assert info0.cycles == co0
    assert np.array_equal(host(X0), xo0)


@pytest.mark.parametrize("tile,s,ov", [((64, 128), 16, (22, 22)), ((64, 128), 12, (22, 22)), ((64, 32), 8, (14, 14))])
def test_4096_benchmark_setting_matches_oracle(orc, tile, s, ov):
    """The benchmark's setting (64 x 128 tiles, s = 16, overlap 22: near the
    exact regime), the exact-regime shape s = 12, overlap 22, and the earlier
    64 x 32 one on the 4096^2 workload: fixed cycles and the solve to 1e-6
    against the oracle."""
    f, h = W.make("poisson2d_4096", 2)
    x0 = np.zeros_like(f)
    say(f"4096^2 fixed 2 cycles T={tile} s={s} o={ov}")
    got, _ = gpu_cycles_2d(f, x0, h, tile, s, 2, ov)
    assert np.array_equal(got, orc.hier_2d(f, x0, h, h, tile, s, 2, ov))
    X = dev(x0)
    say(f"4096^2 solve to 1e-6, T={tile} s={s} o={ov}")
    info = hj.solve_2d(dev(f), X, h, tile=tile, s=s, overlap=ov, rel_tol=1e-6)
    xo, co, relo, _ = orc.solve_2d(f, x0, h, h, tile=tile, s=s, overlap=ov, tol=1e-6, max_cycles=1000)
    assert info.cycles == co
    assert np.array_equal(host(X), xo)
    assert abs(info.rel_residual - relo) <= 1e-12 * relo


# ------------------------------------------------------------------ contracts

def test_resume_equals_one_longer_run():
    f, h = W.make("poisson2d_512", 1)
    a, _ = gpu_cycles_2d(f, np.zeros_like(f), h, (32, 32), 8, 40)
    b, _ = gpu_cycles_2d(f, np.zeros_like(f), h, (32, 32), 8, 20)
    b, _ = gpu_cycles_2d(f, b, h, (32, 32), 8, 20)
    assert np.array_equal(a, b)


def test_not_converged_returns_last_iterate(orc):
    f, h = W.make("poisson2d_512", 0)
    x0 = np.zeros_like(f)
    X = dev(x0)
    info = hj.solve_2d(dev(f), X, h, s=8, rel_tol=1e-12, max_cycles=5, allow_not_converged=True)
    assert info.status == hj.HJ_ERR_NOT_CONVERGED and info.cycles == 5
    want = orc.hier_2d(f, x0, h, h, (32, 32), 8, 5)
    assert np.array_equal(host(X), want)
    _, nr = orc.residual_2d(f, want, h, h)
    _, n0 = orc.residual_2d(f, x0, h, h)
    assert abs(info.rel_residual - nr / n0) <= 1e-12 * (nr / n0)
    with pytest.raises(hj.HJError):
        hj.solve_2d(dev(f), dev(x0), h, s=8, rel_tol=1e-12, max_cycles=3)


def test_nonfinite_rhs_is_reported():
    f = W.rhs_random((64, 64), 1)
    f[10, 20] = np.nan
    with pytest.raises(hj.HJError) as e:
        hj.solve_2d(dev(f), dev(np.zeros_like(f)), 1 / 65, rel_tol=1e-6)
    assert e.value.status == hj.HJ_ERR_NONFINITE


def test_zero_rhs_converges_at_cycle_zero():
    X = dev(np.zeros((64, 64)))
    info = hj.solve_2d(dev(np.zeros((64, 64))), X, 1 / 65, rel_tol=1e-6)
    assert info.cycles == 0 and info.rel_residual == 0.0


def test_host_pointer_is_rejected():
    lib = hj.load()
    a = np.zeros(64 * 64)
    p = hj.make_params()
    info = hj._Info()
    ptr = a.ctypes.data
    st = lib.hj_solve_2d(64, 64, 64, 1 / 65, 1 / 65, 0, ptr, ptr, ctypes.byref(p), None, ctypes.byref(info))
    assert st == hj.HJ_ERR_INVALID_ARG


def test_pitched_rows_leave_padding_untouched(orc):
    ny, nx, ld = 70, 90, 97
    f = W.rhs_random((ny, nx), 71)
    x0 = W.rhs_random((ny, nx), 72)
    h = 1.0 / 91
    Fp = torch.full((ny, ld), 7.0, dtype=torch.float64, device="cuda")
    Xp = torch.full((ny, ld), -3.0, dtype=torch.float64, device="cuda")
    Fp[:, :nx] = dev(f)
    Xp[:, :nx] = dev(x0)
    F, X = Fp[:, :nx], Xp[:, :nx]
    hj.solve_2d(F, X, h, tile=(32, 32), s=5, rel_tol=0.0, max_cycles=3)
    out = host(Xp)
    assert np.array_equal(out[:, :nx], orc.hier_2d(f, x0, h, h, (32, 32), 5, 3))
    assert np.all(out[:, nx:] == -3.0)


def test_side_stream(orc):
    f, h = W.make("poisson2d_512", 2)
    x0 = np.zeros_like(f)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        F, X = dev(f), dev(x0)
        hj.solve_2d(F, X, h, s=4, rel_tol=0.0, max_cycles=6)
    s.synchronize()
    assert np.array_equal(host(X), orc.hier_2d(f, x0, h, h, (32, 32), 4, 6))


# ------------------------------------------------------------------ mixed precision (FP32 cycles, FP64 refinement)

def kappa_2d(n):
    """Condition number of the 5-point Dirichlet Laplacian on an n x n grid:
    lambda_max / lambda_min = cot^2(pi h / 2), h = 1 / (n + 1)."""
    return 1.0 / np.tan(np.pi / (2 * (n + 1))) ** 2


def direct_solve_2d(f, h):
    """A^-1 f for the 5-point Dirichlet Laplacian (sparse LU, independent of
    the oracle and of the GPU path)."""
    import scipy.sparse as sp
    import scipy.sparse.linalg as spla
    ny, nx = f.shape
    def lap(m):
        return sp.diags([-np.ones(m - 1), 2 * np.ones(m), -np.ones(m - 1)], [-1, 0, 1]) / h ** 2
    A = sp.kron(sp.identity(ny), lap(nx)) + sp.kron(lap(ny), sp.identity(nx))
    return spla.spsolve(A.tocsc(), f.ravel()).reshape(ny, nx)


def fp64_residual_np(f, x, h):
    xp = np.pad(x, 1)
    ax = (4 * x - xp[1:-1, :-2] - xp[1:-1, 2:] - xp[:-2, 1:-1] - xp[2:, 1:-1]) / h ** 2
    return np.linalg.norm(f - ax) / np.linalg.norm(f)


@pytest.mark.parametrize("tile,s,ov,seed", [((64, 32), 8, (14, 14), 2), ((64, 32), 8, (14, 14), 3),
                                            ((32, 32), 16, (0, 0), 2)])
def test_refined_solve_reaches_1e10_and_matches_fp64_oracle(orc, tile, s, ov, seed):
    n = 256
    f = W.rhs_2d_modes(n, n, 8, 0.0, seed)
    h = 1.0 / (n + 1)
    X = dev(np.zeros_like(f))
    info = hj.solve_2d_refined(dev(f), X, h, tile=tile, s=s, overlap=ov, rel_tol=1e-10, inner_tol=1e-4,
                               inner_max_cycles=5000, max_outer=12)
    x = host(X)
    rel_np = fp64_residual_np(f, x, h)  # FP64 residual of the result, formed here from the definition
    say(f"refined {tile} s={s} ov={ov} seed={seed}: fp64 cycles={info.fp64_cycles} outer={info.outer} "
        f"inner_cycles={info.inner_cycles} rel={info.rel_residual:.3e} (numpy {rel_np:.3e})")
    assert info.rel_residual <= 1e-10 and rel_np <= 1.001e-10
    assert abs(info.rel_residual - rel_np) <= 1e-3 * rel_np
    # phase 1 is the FP64 solve to 1e5 * rel_tol in the exact regime (overlap
    # >= 2s - 2), else 1e4 * rel_tol; it hands over the iterate one cycle past
    # the oracle's count (computed while the verdict was reached)
    sw = 1e-5 if min(ov) >= 2 * s - 2 else 1e-6
    _, c1, _, _ = orc.solve_2d(f, np.zeros_like(f), h, h, tile=tile, s=s, overlap=ov, tol=sw)
    assert info.fp64_cycles == c1 + 1
    xo, co, relo, _ = orc.solve_2d(f, np.zeros_like(f), h, h, tile=tile, s=s, overlap=ov, tol=1e-10)
    xs = direct_solve_2d(f, h)
    err, err_o = rel(x, xs), rel(xo, xs)
    say(f"  error vs the direct solve: refined {err:.3e}, FP64 oracle solve {err_o:.3e} (both to 1e-10; "
        f"the residuals alone allow kappa*r = {kappa_2d(n) * rel_np:.3e}); refined vs oracle {rel(x, xo):.3e}; "
        f"FP64 cycles {co}")
    # the refined result is as accurate as the FP64 solve to the same
    # tolerance (within a factor 2), far below what its residual alone
    # allows: the error an FP64 step of the refinement done in FP32 leaves
    # (the FP32 rounding of x, ~6e-8) would also exceed it on the overlapped
    # cases, where the FP64 solve's error is ~1e-10
    assert err <= 2.0 * err_o + 1e-13
    # restarting the cycle on the correction equation continues the same
    # iteration (exactly, in exact arithmetic); in FP32 the correction solve
    # gains a little less per cycle near its floor (about eps32 * kappa when
    # the residual sits in the slowest modes, as without overlap)
    total = info.fp64_cycles + info.inner_cycles
    assert abs(total - co) <= 2 * info.outer + 4 + co // 25


@pytest.mark.parametrize("seed,c1", [(0, 3), (5, 7)])
def test_refined_solve_stays_fp64_when_the_switch_point_comes_early(orc, seed, c1):
    """The FP64 cycles reach the switch point (1e5 * rel_tol in the exact
    regime) in c1 < 8 cycles: no hand-over, the result is hj_solve_2d's FP64
    solve to rel_tol bit for bit (equal to the oracle's), outer = 0.  With
    switch_min_cycles = 1 the same problem hands over at cycle c1 and
    refines."""
    n = 256
    f = W.rhs_2d_modes(n, n, 8, 0.0, seed)
    h = 1.0 / (n + 1)
    kw = dict(tile=(64, 32), s=8, overlap=(14, 14))
    _, c1o, _, _ = orc.solve_2d(f, np.zeros_like(f), h, h, tol=1e-5, **kw)
    assert c1o == c1
    X = dev(np.zeros_like(f))
    info = hj.solve_2d_refined(dev(f), X, h, rel_tol=1e-10, inner_tol=1e-6, **kw)
    Y = dev(np.zeros_like(f))
    one = hj.solve_2d(dev(f), Y, h, rel_tol=1e-10, **kw)
    xo, co, _, _ = orc.solve_2d(f, np.zeros_like(f), h, h, tol=1e-10, **kw)
    say(f"refined seed {seed}: outer {info.outer}, fp64 cycles {info.fp64_cycles} (FP64 solve {one.cycles})")
    assert info.outer == 0 and info.inner_cycles == 0
    assert info.fp64_cycles == one.cycles == co
    assert torch.equal(X, Y) and np.array_equal(host(X), xo)
    assert info.rel_residual == one.rel_residual
    X.zero_()
    forced = hj.solve_2d_refined(dev(f), X, h, rel_tol=1e-10, inner_tol=1e-6, switch_min_cycles=1, **kw)
    assert forced.outer >= 1 and forced.fp64_cycles == c1 + 1
    assert fp64_residual_np(f, host(X), h) <= 1.001e-10


def test_refined_solve_fp32_from_the_start_still_converges():
    """switch_tol >= 1: refinement alone (no FP64 phase) reaches 1e-10; FP32
    rounding leaves slow-mode error that costs extra cycles, which is why the
    default starts FP32 only near rel_tol * 1e4."""
    n = 128
    f = W.rhs_2d_modes(n, n, 8, 0.0, 5)
    h = 1.0 / (n + 1)
    X = dev(np.zeros_like(f))
    info = hj.solve_2d_refined(dev(f), X, h, tile=(32, 32), s=8, overlap=(14, 14), rel_tol=1e-10,
                               inner_tol=1e-4, switch_tol=1.0, inner_max_cycles=20000, max_outer=20)
    rel_np = fp64_residual_np(f, host(X), h)
    say(f"refined from FP32 start: outer={info.outer} inner={info.inner_cycles} rel={rel_np:.3e}")
    assert info.fp64_cycles == 0 and info.outer >= 1
    assert info.rel_residual <= 1e-10 and rel_np <= 1.001e-10


def test_refined_solve_reports_not_converged():
    f = W.rhs_2d_modes(128, 128, 8, 0.0, 1)
    X = dev(np.zeros_like(f))
    info = hj.solve_2d_refined(dev(f), X, 1 / 129, tile=(32, 32), s=4, overlap=(0, 0), rel_tol=1e-12,
                               inner_tol=1e-2, switch_tol=1.0, max_outer=2, allow_not_converged=True)
    assert info.status == hj.HJ_ERR_NOT_CONVERGED and info.outer == 2
    with pytest.raises(hj.HJError):
        hj.solve_2d_refined(dev(f), dev(np.zeros_like(f)), 1 / 129, tile=(32, 32), s=4,
                            overlap=(0, 0), rel_tol=1e-12, inner_tol=1e-2, switch_tol=1.0, max_outer=2)


# ------------------------------------------------------------------ FP32 instantiation

def test_fp32_iterates_within_1e5_of_fp64_oracle(orc):
    f, h = W.make("poisson2d_512", 0)
    x0 = np.zeros_like(f)
    for s, nc in ((16, 64), (4, 200)):
        got, _ = gpu_cycles_2d(f, x0, h, (32, 32), s, nc, dtype=torch.float32)
        want = orc.hier_2d(f, x0, h, h, (32, 32), s, nc)
        e = rel(got, want)
        say(f"fp32 512^2 s={s} cycles={nc}: rel err vs fp64 oracle {e:.3e}")
        assert e <= 1e-5
    n = 1000
    f1 = W.rhs_1d_modes(n, 8, 1)
    got, _ = gpu_cycles_1d(f1, np.zeros(n), 1 / (n + 1), 64, 16, 50, dtype=torch.float32)
    assert rel(got, orc.hier_1d(f1, np.zeros(n), 1 / (n + 1), 64, 16, 50)) <= 1e-5


# ------------------------------------------------------------------ the shape for grids of few tiles

@pytest.mark.parametrize("tile,n", [((32, 16), (40, 18)), ((32, 32), (33, 32)), ((32, 64), (100, 70)), ((32, 128), (64, 129)),
                                    ((64, 16), (64, 16)), ((64, 32), (70, 65)), ((64, 64), (129, 64)), ((64, 128), (64, 130)),
                                    ((32, 32), (1024, 1024)), ((32, 32), (1056, 1024))])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("iso", [True, False])
def test_few_tiles_shape_matches_oracle(orc, tile, n, dtype, iso):
    """Grids of one to a few tiles run two rows a lane, with their own order of
    loads and flag; 1024^2 and 1056 x 1024 with 32 x 32 tiles lie on either
    side of the rule.  Cycles that fuse the residual, and cycles that do not."""
    nx, ny = n
    f, x0 = W.rhs_random((ny, nx), 21), W.rhs_random((ny, nx), 22)
    hx = 1.0 / (nx + 1)
    hy = hx if iso else 1.3 * hx
    hier = orc.hier_2d if dtype == torch.float64 else orc.hier_2d_f32
    for s, ov, nc in ((1, (0, 0), 3), (4, (6, 6), 2), (5, (3, 2), 3)):
        say(f"few tiles {tile} {n} {dtype} iso={iso} s={s}")
        want = hier(f, x0, hx, hy, tile, s, nc, ov)
        for tol in (0.0, 1e-100):
            F, X = dev(f, dtype), dev(x0, dtype)
            info = hj.solve_2d(F, X, hx=hx, hy=hy, tile=tile, s=s, overlap=ov, rel_tol=tol, max_cycles=nc,
                               allow_not_converged=True)
            assert info.cycles == nc
            assert np.array_equal(host(X), want), (s, ov, tol)


@pytest.mark.parametrize("n,tile,ov", [((5003, 3301), (32, 32), (6, 2)), ((2600, 6007), (64, 128), (22, 22))])
def test_strip_walk_reaches_every_tile(orc, n, tile, ov):
    """Grids large enough to be walked in strips, ragged, the last strip narrower than the others."""
    nx, ny = n
    f, x0 = W.rhs_random((ny, nx), 31), W.rhs_random((ny, nx), 32)
    h = 1.0 / (nx + 1)
    say(f"strip walk {n} {tile} {ov}")
    got, _ = gpu_cycles_2d(f, x0, h, tile, 2, 2, ov)
    assert np.array_equal(got, orc.hier_2d(f, x0, h, h, tile, 2, 2, ov))


@pytest.mark.parametrize("method", ["hierarchical", "global"])
def test_stop_is_the_same_however_often_the_host_looks(orc, method):
    """Solves that stop at iterate 0, 1, 2, ... and at the last one, with the host's
    own batches, a look after every cycle, batches past the stop, and without
    pinned memory (the allocation-free entry)."""
    nx, ny = 90, 70
    hx, hy = 1.0 / (nx + 1), 1.2 / (nx + 1)
    rng = np.random.default_rng(11)
    f, x0 = rng.standard_normal((ny, nx)), 1e-3 * rng.standard_normal((ny, nx))
    kw = dict(hx=hx, hy=hy, tile=(32, 32), s=4, overlap=(6, 6), method=method, allow_not_converged=True)
    rel = []
    for k in range(24):
        X = dev(x0)
        rel.append(hj.solve_2d(dev(f), X, rel_tol=0.0, max_cycles=k, **kw).rel_residual if k else 1.0)
    for want in [k for k in range(24) if all(rel[k] < r * (1 - 1e-9) for r in rel[:k])]:
        tol = rel[want] * (1 + 1e-10)
        X = dev(x0)
        ref = hj.solve_2d(dev(f), X, rel_tol=0.0, max_cycles=max(want, 1), **kw)
        ref = host(X) if want else x0
        for solve, every, cap in ((hj.solve_2d, 0, 1000), (hj.solve_2d, 1, 1000), (hj.solve_2d, 500, 1000),
                                  (hj.solve_2d, 0, max(want, 1)), (hj.solve_2d_noalloc, 0, 1000)):
            X = dev(x0)
            info = solve(dev(f), X, rel_tol=tol, max_cycles=cap, check_every=every, **kw)
            assert info.cycles == want and info.status == hj.HJ_OK, (want, every, cap)
            assert np.array_equal(host(X), ref), (want, every, cap)


@pytest.mark.parametrize("n,tile,ov", [((4263, 4263), (32, 32), (6, 2)), ((4264, 4264), (32, 32), (2, 6)),
                                       ((2602, 9001), (64, 128), (22, 22)), ((5003, 4999), (32, 32), (2, 6))])
def test_fp32_walk_on_both_sides_of_the_strip_rule(orc, n, tile, ov):
    """FP32 grids just below and above the size from which they are walked in strips."""
    nx, ny = n
    f, x0 = W.rhs_random((ny, nx), 41), W.rhs_random((ny, nx), 42)
    h = 1.0 / (nx + 1)
    say(f"fp32 walk {n} {tile} {ov}")
    got, _ = gpu_cycles_2d(f, x0, h, tile, 2, 2, ov, dtype=torch.float32)
    assert np.array_equal(got, orc.hier_2d_f32(f, x0, h, h, tile, 2, 2, ov))


@pytest.mark.parametrize("n", [(32 * 64, 128 * 32), (32 * 63 - 5, 128 * 32 - 3), (32 * 63, 128 * 32)])
@pytest.mark.parametrize("iso", [True, False])
def test_many_tiles_shape_matches_oracle(orc, n, iso):
    """FP64 32 x 128 tiles on both sides of 2048 of them (2048, 2016 and 2016), with and without residual."""
    nx, ny = n
    f, x0 = W.rhs_random((ny, nx), 51), W.rhs_random((ny, nx), 52)
    hx = 1.0 / (nx + 1)
    hy = hx if iso else 1.3 * hx
    for s, ov in ((1, (0, 0)), (4, (3, 6)), (5, (0, 0))):
        say(f"many tiles {n} iso={iso} s={s}")
        want = orc.hier_2d(f, x0, hx, hy, (32, 128), s, 2, ov)
        for tol in (0.0, 1e-100):
            X = dev(x0)
            hj.solve_2d(dev(f), X, hx=hx, hy=hy, tile=(32, 128), s=s, overlap=ov, rel_tol=tol, max_cycles=2,
                        allow_not_converged=True)
            assert np.array_equal(host(X), want), (s, ov, tol)


# ------------------------------------------------------------------ cycles of more than 2^32 threads

@pytest.mark.parametrize("n,tile,ov,lds", [((5860, 5850), (32, 32), (31, 31), False), ((4130, 4120), (16, 16), (15, 15), True),
                                           ((4150, 4200), (32, 64), (31, 63), False)])
def test_cycles_of_more_threads_than_a_launch_counts(n, tile, ov, lds):
    """Tiles a point apart: with s = 1 a cycle is one classical sweep, whatever their number."""
    nx, ny = n
    tiles = hj.axis_tiles(nx, tile[0], ov[0]) * hj.axis_tiles(ny, tile[1], ov[1])
    assert tiles * (256 if lds else 4 * tile[1]) > 2 ** 32
    gen = torch.Generator(device="cuda").manual_seed(7)
    f = torch.randn(ny, nx, dtype=torch.float64, device="cuda", generator=gen)
    x0 = torch.randn(ny, nx, dtype=torch.float64, device="cuda", generator=gen)
    h = 1.0 / (nx + 1)
    say(f"threads {n} {tile} o={ov}")
    for tol in (0.0, 1e-100):
        kw = dict(rel_tol=tol, max_cycles=3, allow_not_converged=True)
        X, Y = x0.clone(), x0.clone()
        info = hj.solve_2d(f, X, h, tile=tile, s=1, overlap=ov, lds_kernel=lds, **kw)
        ref = hj.solve_2d(f, Y, h, method="global", **kw)
        assert torch.equal(X, Y), tol
        # sums of 3.4e7 squares in two orders, each by at least 15 levels of partial sums
        assert abs(info.r0_norm - ref.r0_norm) <= 1e-11 * ref.r0_norm
        assert abs(info.rel_residual - ref.rel_residual) <= 2e-11 * ref.rel_residual


def test_batch_of_more_threads_than_a_launch_counts():
    n, ov = 4140, 31
    assert 2 * hj.axis_tiles(n, 32, ov) ** 2 * 128 > 2 ** 32
    gen = torch.Generator(device="cuda").manual_seed(8)
    f = torch.randn(2, n, n, dtype=torch.float64, device="cuda", generator=gen)
    X = torch.zeros_like(f)
    say("threads, batch")
    hj.solve_batched([(f[i], X[i], 1.0 / (n + 1)) for i in range(2)], rel_tol=0.0, tile=(32, 32), s=1, overlap=(ov, ov),
                     max_cycles=3)
    for i in range(2):
        Y = torch.zeros_like(f[i])
        hj.solve_2d(f[i], Y, 1.0 / (n + 1), method="global", rel_tol=0.0, max_cycles=3)
        assert torch.equal(X[i], Y), i


def test_1d_cycles_of_more_threads_than_a_launch_counts_are_refused():
    n = 2 ** 26 + 2 ** 10
    f = torch.zeros(n, dtype=torch.float32, device="cuda")
    with pytest.raises(hj.HJError):
        hj.solve_1d(f, torch.zeros_like(f), 1.0 / (n + 1), tile=64, s=1, overlap=63, rel_tol=0.0, max_cycles=1)
