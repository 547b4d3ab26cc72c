"""GPU parity for variable-coefficient diffusion -div(a grad u) = f and its
adjoint: forward iterates and cycles-to-tolerance against the CPU oracle, the
gradient with respect to a against the oracle's face-product formula (itself
pinned by finite differences of direct solves), and torch autograd through the
adjoint solve against central finite differences."""
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


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).to(dtype=torch.float64, device="cuda")


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.fixture(scope="module")
def prob():
    ny, nx = 48, 64
    hx, hy = 1.0 / (nx + 1), 1.0 / (ny + 1)
    a = np.exp(W.grf_2d(ny + 2, nx + 2, 0.15, 1.0, hx, seed=7))
    f = np.stack([W.rhs_2d_modes(nx, ny, 8, 0.1, s) for s in range(3)])
    return nx, ny, hx, hy, a, f


# 64 x 48 grid: the first four shapes hold a full tile in each direction and
# run register-resident tiles by default; (16, 64) and (32, 64) are taller
# than the grid and run the LDS tile.  lds_kernel forces the LDS tile.
@pytest.mark.parametrize("lds", [False, True], ids=["default", "lds"])
@pytest.mark.parametrize("tile,s,ov", [((32, 32), 8, (0, 0)), ((16, 16), 4, (6, 6)), ((64, 16), 3, (2, 2)),
                                       ((64, 32), 8, (14, 14)), ((16, 64), 5, (8, 8)), ((32, 64), 2, (0, 0))])
def test_vc_fixed_cycles_match_oracle(orc, prob, tile, s, ov, lds):
    nx, ny, hx, hy, a, f = prob
    U = torch.zeros_like(dev(f))
    hj.solve_vc_2d(dev(a), dev(f), U, hx=hx, hy=hy, tile=tile, s=s, overlap=ov, rel_tol=0.0, max_cycles=5,
                   lds_kernel=lds)
    got = host(U)
    for b in range(f.shape[0]):
        want = orc.vc_solve_2d(a, f[b], np.zeros((ny, nx)), hx, hy, tile=tile, s=s, overlap=ov,
                               tol=0.0, max_cycles=5)[0]
        assert np.array_equal(got[b], want), f"batch {b}"


@pytest.mark.parametrize("tile,s,ov", [((64, 32), 8, (14, 14)), ((32, 64), 6, (10, 10)), ((16, 32), 3, (0, 0)),
                                       ((64, 64), 4, (6, 6))])
def test_vc_register_tiles_on_a_ragged_grid_match_oracle(orc, tile, s, ov):
    """150 x 75 with anisotropic spacing: several tiles per axis with the
    last one moved left to end at the grid edge, so the ownership split
    between overlapping tiles is uneven; register-resident tiles (default)
    and the LDS tile must both give the oracle's iterates bit for bit, after
    fixed cycles and at the tolerance (the residual fused into the load)."""
    nx, ny = 150, 75
    hx, hy = 1.0 / (nx + 1), 1.3 / (ny + 1)
    a = np.exp(W.grf_2d(ny + 2, nx + 2, 0.1, 1.0, hx, seed=3))
    f = np.stack([W.rhs_2d_modes(nx, ny, 8, 0.1, 40 + b) for b in range(2)])
    x0 = np.stack([W.rhs_random((ny, nx), 50 + b) for b in range(2)])
    kw = dict(tile=tile, s=s, overlap=ov)
    for lds in (False, True):
        U = dev(x0)
        hj.solve_vc_2d(dev(a), dev(f), U, hx=hx, hy=hy, rel_tol=0.0, max_cycles=3, lds_kernel=lds, **kw)
        got = host(U)
        for b in range(2):
            want = orc.vc_solve_2d(a, f[b], x0[b], hx, hy, tol=0.0, max_cycles=3, **kw)[0]
            assert np.array_equal(got[b], want), f"lds={lds} b={b} fixed cycles"
    U = dev(x0)
    infos = hj.solve_vc_2d(dev(a), dev(f), U, hx=hx, hy=hy, rel_tol=1e-7, **kw)
    got = host(U)
    for b in range(2):
        xo, co, relo, _ = orc.vc_solve_2d(a, f[b], x0[b], hx, hy, tol=1e-7, **kw)
        say(f"vc ragged {tile} s={s} b={b}: gpu cycles {infos[b].cycles}, oracle {co}")
        assert infos[b].cycles == co
        assert np.array_equal(got[b], xo)
        assert abs(infos[b].rel_residual - relo) <= 1e-9 * relo


def test_vc_classical_and_tolerance_match_oracle(orc, prob):
    nx, ny, hx, hy, a, f = prob
    U = torch.zeros_like(dev(f))
    hj.solve_vc_2d(dev(a), dev(f), U, hx=hx, hy=hy, method="global", rel_tol=0.0, max_cycles=17)
    for b in range(f.shape[0]):
        want = orc.vc_solve_2d(a, f[b], np.zeros((ny, nx)), hx, hy, method=orc.CLASSICAL, tol=0.0,
                               max_cycles=17)[0]
        assert np.array_equal(host(U)[b], want)
    U.zero_()
    infos = hj.solve_vc_2d(dev(a), dev(f), U, hx=hx, hy=hy, tile=(32, 32), s=8, overlap=(14, 14),
                           rel_tol=1e-8)
    for b in range(f.shape[0]):
        xo, co, relo, _ = orc.vc_solve_2d(a, f[b], np.zeros((ny, nx)), hx, hy, tile=(32, 32), s=8,
                                          overlap=(14, 14), tol=1e-8)
        say(f"vc solve b={b}: gpu cycles {infos[b].cycles}, oracle {co}")
        assert infos[b].cycles == co
        assert np.array_equal(host(U)[b], xo)
        assert abs(infos[b].rel_residual - relo) <= 1e-9 * relo


def test_vc_batch_equals_single_rhs_solves(prob):
    """Several right-hand sides run through the batched engine; each must end
    where its own single-right-hand-side solve ends: same iterate bit for
    bit, same cycle count, also when some stop at max_cycles."""
    nx, ny, hx, hy, a, f = prob
    opts = dict(hx=hx, hy=hy, tile=(16, 32), s=6, overlap=(10, 10))
    for tol, cap in ((1e-9, 1_000_000), (1e-9, 40)):
        U = torch.zeros_like(dev(f))
        infos = hj.solve_vc_2d(dev(a), dev(f), U, rel_tol=tol, max_cycles=cap, allow_not_converged=True, **opts)
        for b in range(f.shape[0]):
            Ub = torch.zeros_like(dev(f[b:b + 1]))
            one = hj.solve_vc_2d(dev(a), dev(f[b:b + 1]), Ub, rel_tol=tol, max_cycles=cap,
                                 allow_not_converged=True, **opts)[0]
            say(f"vc batch b={b} cap={cap}: batched {infos[b].cycles} single {one.cycles}")
            assert infos[b].cycles == one.cycles <= cap
            assert np.array_equal(host(U)[b], host(Ub)[0])
            assert abs(infos[b].rel_residual - one.rel_residual) <= 1e-12 * one.rel_residual
            assert (infos[b].rel_residual <= tol) == (one.rel_residual <= tol)


def test_vc_gradient_matches_oracle_formula(orc, prob):
    nx, ny, hx, hy, a, f = prob
    u = np.stack([W.rhs_random((ny, nx), 20 + b) for b in range(3)])
    lam = np.stack([W.rhs_random((ny, nx), 30 + b) for b in range(3)])
    g = host(hj.vc_grad_a(dev(a), dev(u), dev(lam), hx=hx, hy=hy))
    want = sum(orc.vc_grad_a_2d(u[b], lam[b], hx, hy) for b in range(3))
    assert np.max(np.abs(g - want)) <= 1e-12 * np.max(np.abs(want))


def test_adjoint_solve_and_autograd_against_finite_differences(orc):
    ny, nx = 20, 24
    hx, hy = 1.0 / (nx + 1), 1.0 / (ny + 1)
    a0 = np.exp(W.grf_2d(ny + 2, nx + 2, 0.2, 1.0, hx, seed=11))
    f0 = np.stack([W.rhs_2d_modes(nx, ny, 6, 0.0, s) for s in range(2)])
    t = np.stack([W.smooth_modes_2d(nx, 3, 3, s)[:ny, :] for s in range(2)]) * 1e-3
    opts = dict(hx=hx, hy=hy, tile=(16, 16), s=6, overlap=(10, 10), rel_tol=1e-13)
    T = dev(t)

    def loss_of(A, F):
        return torch.mean((hj.diffusion_solve(F, A, **opts) - T) ** 2)

    A = dev(a0).requires_grad_(True)
    F = dev(f0).requires_grad_(True)
    L = loss_of(A, F)
    L.backward()
    ga, gf = host(A.grad), host(F.grad)

    # against the oracle: same solves on the CPU, adjoint formula for dL/da
    us = [orc.vc_solve_2d(a0, f0[b], np.zeros((ny, nx)), hx, hy, tile=(16, 16), s=6, overlap=(10, 10),
                          tol=1e-13)[0] for b in range(2)]
    n = t.size
    lams = [orc.vc_solve_2d(a0, 2 * (us[b] - t[b]) / n, np.zeros((ny, nx)), hx, hy, tile=(16, 16), s=6,
                            overlap=(10, 10), tol=1e-13)[0] for b in range(2)]
    want_ga = sum(orc.vc_grad_a_2d(us[b], lams[b], hx, hy) for b in range(2))
    assert np.max(np.abs(ga - want_ga)) <= 1e-8 * np.max(np.abs(want_ga))
    assert np.max(np.abs(gf - np.stack(lams))) <= 1e-8 * np.max(np.abs(gf))

    # central finite differences (eps = 1e-6, FP64) of the GPU forward solve
    rng = np.random.default_rng(3)
    eps = 1e-6
    with torch.no_grad():
        for _ in range(8):
            r, q = rng.integers(0, ny + 2), rng.integers(0, nx + 2)
            Ap, Am = dev(a0), dev(a0)
            Ap[r, q] += eps
            Am[r, q] -= eps
            fd = (loss_of(Ap, dev(f0)) - loss_of(Am, dev(f0))).item() / (2 * eps)
            say(f"dL/da[{r},{q}]: autograd {ga[r, q]:.6e} fd {fd:.6e}")
            assert abs(fd - ga[r, q]) <= 1e-4 * np.max(np.abs(ga)) + 1e-6 * abs(ga[r, q])
        for _ in range(4):
            b, r, q = rng.integers(0, 2), rng.integers(0, ny), rng.integers(0, nx)
            Fp, Fm = dev(f0), dev(f0)
            Fp[b, r, q] += eps
            Fm[b, r, q] -= eps
            fd = (loss_of(dev(a0), Fp) - loss_of(dev(a0), Fm)).item() / (2 * eps)
            assert abs(fd - gf[b, r, q]) <= 1e-4 * np.max(np.abs(gf))


@pytest.mark.parametrize("mode", ["fixed", "tol"])
def test_solve_adjoint_c_abi_pitched_batch(orc, mode):
    """hj_solve_adjoint called through the C ABI on a batch of 3 right-hand
    sides in pitched storage: f/u/lam rows of ld > nx, a batch stride beyond
    ny * ld, coefficient rows of lda > nx + 2 and gradient rows of
    ld_grad > nx + 2, starting from a nonzero guess.  lam equals the oracle's
    solve of dL/du bit for bit (fixed cycles; to tolerance also the cycle
    counts), dL/da equals the oracle's face-product gradient summed over the
    batch within 1e-12, and no padding element is written (NaN padding in the
    inputs would also show any read of it in the results)."""
    ny, nx, B = 40, 56, 3
    ld, lda, ldg = nx + 5, nx + 2 + 3, nx + 2 + 6
    bstride = ny * ld + 37
    hx, hy = 1.0 / (nx + 1), 1.0 / (ny + 1)
    a = np.exp(W.grf_2d(ny + 2, nx + 2, 0.15, 1.0, hx, seed=5))
    u = [W.rhs_random((ny, nx), 40 + b) for b in range(B)]
    dl = [W.rhs_2d_modes(nx, ny, 6, 0.1, 50 + b) for b in range(B)]
    lam0 = [W.rhs_random((ny, nx), 60 + b) * 1e-3 for b in range(B)]

    def flat(arrs, fill):
        buf = np.full(B * bstride, fill)
        for b, arr in enumerate(arrs):
            buf[b * bstride: b * bstride + ny * ld].reshape(ny, ld)[:, :nx] = arr
        return buf

    def unflat(buf):
        return [buf[b * bstride: b * bstride + ny * ld].reshape(ny, ld)[:, :nx] for b in range(B)]

    A = np.full((ny + 2, lda), np.nan)
    A[:, :nx + 2] = a
    dA, dU, dDL = dev(A), dev(flat(u, np.nan)), dev(flat(dl, np.nan))
    LAM = dev(flat(lam0, -7.0))
    G = dev(np.full((ny + 2, ldg), -9.0))
    kw = dict(tile=(32, 16), s=5, overlap=(8, 6))
    tol, cycles = (0.0, 7) if mode == "fixed" else (1e-9, 1_000_000)

    pr = hj.VCProblem()
    pr.nx, pr.ny, pr.ld, pr.lda, pr.hx, pr.hy = nx, ny, ld, lda, hx, hy
    pr.a, pr.batch, pr.flags, pr.batch_stride = dA.data_ptr(), B, 0, bstride
    d = hj.AdjointDesc()
    d.prob = pr
    d.u, d.dl_du, d.lam, d.dl_da, d.ld_grad = dU.data_ptr(), dDL.data_ptr(), LAM.data_ptr(), G.data_ptr(), ldg
    d.params = hj.make_params(kw["tile"], kw["s"], "hierarchical", tol, cycles, 0, kw["overlap"])
    infos = (hj._Info * B)()
    torch.cuda.synchronize()
    st = hj.load().hj_solve_adjoint(ctypes.byref(d), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream),
                                    infos)
    assert st == hj.HJ_OK, hj.last_error()
    lam_buf = host(LAM)
    lams = unflat(lam_buf)
    for b in range(B):
        xo, co, relo, _ = orc.vc_solve_2d(a, dl[b], lam0[b], hx, hy, tile=kw["tile"], s=kw["s"],
                                          overlap=kw["overlap"], tol=tol, max_cycles=cycles)
        say(f"adjoint {mode} b={b}: gpu cycles {infos[b].cycles}, oracle {co}")
        assert np.array_equal(lams[b], xo), f"batch {b}"
        if mode == "tol":
            assert infos[b].cycles == co and abs(infos[b].rel_residual - relo) <= 1e-9 * relo
    # padding of lam untouched
    mask = np.ones(B * bstride, bool)
    for b in range(B):
        mask[b * bstride: b * bstride + ny * ld].reshape(ny, ld)[:, :nx] = False
    assert np.all(lam_buf[mask] == -7.0)
    g = host(G)
    want = sum(orc.vc_grad_a_2d(u[b], lams[b], hx, hy) for b in range(B))
    assert np.all(g[:, nx + 2:] == -9.0)
    assert np.max(np.abs(g[:, :nx + 2] - want)) <= 1e-12 * np.max(np.abs(want))


def test_solve_adjoint_binding_without_gradient(orc, prob):
    """The binding's solve_adjoint with grad_a=False passes NULL dl_da: lam is
    the adjoint solve alone and no gradient is formed."""
    nx, ny, hx, hy, a, f = prob
    Lam = torch.zeros_like(dev(f))
    infos, g = hj.solve_adjoint(dev(a), None, dev(f), Lam, hx=hx, hy=hy, tile=(32, 32), s=8, overlap=(14, 14),
                                rel_tol=0.0, max_cycles=4, grad_a=False)
    assert g is None and len(infos) == f.shape[0]
    for b in range(f.shape[0]):
        want = orc.vc_solve_2d(a, f[b], np.zeros((ny, nx)), hx, hy, tile=(32, 32), s=8, overlap=(14, 14),
                               tol=0.0, max_cycles=4)[0]
        assert np.array_equal(host(Lam)[b], want)


def test_vc_config_size_forward_and_adjoint_match_oracle(orc):
    """The differentiable configuration at its own size: 1024 x 1024,
    a = exp(g) (squared-exponential field, length 0.05, variance 1), 16
    right-hand sides through the batched engine.  Three fixed cycles of the
    forward solve (64 x 32 tiles, s = 8, overlap 14) equal the oracle's per
    right-hand side bit for bit; the adjoint solve through hj_solve_adjoint
    on dL/du = 2 (u - t) / N from those states equals the oracle's solve of
    the same right-hand sides bit for bit, and dL/da equals the oracle's
    face-product gradient summed over the batch within 1e-12."""
    n, B, K = 1024, 16, 3
    h = 1.0 / (n + 1)
    kw = dict(tile=(64, 32), s=8, overlap=(14, 14))
    a = W.diffusion_coefficient(n, 0.05, 1.0, 7)
    f = np.stack([W.rhs_2d_modes(n, n, 8, 0.0, b) for b in range(B)])
    A, F = dev(a), dev(f)
    U = torch.zeros_like(F)
    hj.solve_vc_2d(A, F, U, h, rel_tol=0.0, max_cycles=K, **kw)
    u = host(U)
    for b in range(B):
        want = orc.vc_solve_2d(a, f[b], np.zeros((n, n)), h, h, tol=0.0, max_cycles=K, **kw)[0]
        assert np.array_equal(u[b], want), f"forward, right-hand side {b}"
    t = np.stack([W.smooth_modes_2d(n, 3, 3, 100 + b) for b in range(B)]) * 1e-3
    dl = 2.0 * (u - t) / u.size
    LAM = torch.zeros_like(F)
    infos, G = hj.solve_adjoint(A, U, dev(dl), LAM, h, rel_tol=0.0, max_cycles=K, **kw)
    lam = host(LAM)
    assert len(infos) == B and all(i.cycles == K for i in infos)
    for b in range(B):
        want = orc.vc_solve_2d(a, dl[b], np.zeros((n, n)), h, h, tol=0.0, max_cycles=K, **kw)[0]
        assert np.array_equal(lam[b], want), f"adjoint, right-hand side {b}"
    want_g = sum(orc.vc_grad_a_2d(u[b], lam[b], h, h) for b in range(B))
    g = host(G)
    err = np.max(np.abs(g - want_g)) / np.max(np.abs(want_g))
    say(f"1024^2 x 16: dL/da max difference {err:.2e} of the largest entry")
    assert err <= 1e-12


@pytest.mark.parametrize("n,tile,ov", [((3000, 2503), (64, 32), (14, 14)), ((130, 97), (64, 64), (6, 4)),
                                       ((64, 64), (64, 64), (0, 0)), ((33, 47), (32, 32), (5, 3)), ((40, 64), (64, 32), (2, 2))])
@pytest.mark.parametrize("s", [1, 2, 5])
def test_vc_cycle_bodies_match_oracle(orc, n, tile, ov, s):
    """A grid walked in strips, whole and ragged register tiles, a grid below the tile
    (LDS body); odd and even sub-iterations (two per loop trip)."""
    nx, ny = n
    if nx > 1000 and s != 2:
        pytest.skip("one sub-iteration count at the large size")
    hx, hy = 1.0 / (nx + 1), 1.2 / (nx + 1)
    rng = np.random.default_rng(3)
    a = np.exp(0.5 * rng.standard_normal((ny + 2, nx + 2)))
    f, u0 = rng.standard_normal((ny, nx)), rng.standard_normal((ny, nx))
    say(f"vc bodies {n} {tile} {ov} s={s}")
    nc = 2
    want = orc.vc_solve_2d(a, f, u0, hx, hy, tile=tile, s=s, tol=-1.0, max_cycles=nc, overlap=ov)[0]
    for lds in (False, True):
        for tol in (0.0, 1e-100):
            U = dev(u0)
            hj.solve_vc_2d(dev(a), dev(f), U, hx=hx, hy=hy, tile=tile, s=s, overlap=ov, rel_tol=tol, max_cycles=nc,
                           allow_not_converged=True, lds_kernel=lds)
            assert np.array_equal(host(U), want), (lds, tol)


# heights on both sides of every row count a wavefront (16, 24, 32, 48, 64),
# widths below and at 64, and one step past the one-workgroup solve (65)
@pytest.mark.parametrize("nx,ny", [(64, 64), (63, 64), (64, 63), (1, 1), (3, 2), (64, 16), (40, 17), (64, 24), (33, 25),
                                   (64, 32), (17, 33), (64, 48), (5, 49), (65, 20), (20, 65)])
@pytest.mark.parametrize("s", [1, 2, 3, 8])
def test_vc_one_workgroup_solves_match_oracle(orc, nx, ny, s):
    rng = np.random.default_rng(nx + 100 * ny + s)
    hx, hy = 1.0 / (nx + 1), 0.9 / (ny + 1)
    a = np.exp(0.5 * rng.standard_normal((ny + 2, nx + 2)))
    f, u0 = rng.standard_normal((3, ny, nx)), rng.standard_normal((3, ny, nx))
    kw = dict(tile=(32, 32), s=s, overlap=(2 * s - 2, 2 * s - 1))
    say(f"vc one workgroup {nx} x {ny} s={s}")
    for nb in (1, 3):
        for tol, cap in ((0.0, 5), (1e-100, 4), (0.3, 10_000)):
            U = dev(u0[:nb])
            infos = hj.solve_vc_2d(dev(a), dev(f[:nb]), U, hx=hx, hy=hy, rel_tol=tol, max_cycles=cap,
                                   allow_not_converged=True, **kw)
            got = host(U)
            for b in range(nb):
                xo, co, relo, r0o = orc.vc_solve_2d(a, f[b], u0[b], hx, hy, tol=tol, max_cycles=cap, **kw)
                assert np.array_equal(got[b], xo), (nb, b, tol)
                assert infos[b].cycles == (co if co >= 0 else cap)
                # the norms' sums run in another order than the oracle's, over
                # at most 65 x 64 squares: 4160 x 2^-53 of each, on either side
                assert abs(infos[b].r0_norm - r0o) <= 1e-12 * r0o
                assert abs(infos[b].rel_residual - relo) <= 2e-12 * relo


@pytest.mark.parametrize("nx,ny", [(64, 64), (61, 45)])
def test_vc_one_workgroup_not_finite_and_long_runs(nx, ny):
    """Where a solve stops and what it holds when values overflow or are NaN, and
    over more cycles than one launch runs, as by the tile kernels."""
    rng = np.random.default_rng(5)
    h = 1.0 / (nx + 1)
    a = np.exp(rng.standard_normal((ny + 2, nx + 2)))
    f, u0 = rng.standard_normal((2, ny, nx)), rng.standard_normal((2, ny, nx))
    bad = u0.copy()
    bad[0, 7, nx - 1], bad[1, ny - 1, 3] = np.inf, np.nan
    big = u0 * 1e150
    big[:, ny - 1, nx - 1] = -1e160
    for name, x0, tol, cap, s in (("inf", bad, 0.0, 3, 4), ("inf", bad, 1e-9, 9, 4), ("overflow", big, 0.0, 3, 4),
                                  ("long", u0, 0.0, 4200, 1), ("long", u0, 1e-100, 4200, 1)):
        for nb in (1, 2):
            say(f"vc one workgroup {name} {nx} x {ny} tol={tol} x{nb}")
            out = []
            for lds in (False, True):
                U = dev(x0[:nb])
                try:
                    infos = hj.solve_vc_2d(dev(a), dev(f[:nb]), U, hx=h, hy=h, tile=(64, 32), s=s, overlap=(0, 14),
                                           rel_tol=tol, max_cycles=cap, allow_not_converged=True, lds_kernel=lds)
                    st = [(i.status, i.cycles) for i in infos]
                except hj.HJError as e:
                    st = str(e)
                out.append((st, host(U)))
            assert out[0][0] == out[1][0], name
            assert np.array_equal(out[0][1], out[1][1], equal_nan=True), name


def test_vc_one_workgroup_long_cycles_match_oracle(orc):
    """Cycles of more sweeps than a launch runs (one a launch), and of half as many."""
    rng = np.random.default_rng(2)
    a, f = np.exp(0.3 * rng.standard_normal((7, 8))), rng.standard_normal((2, 5, 6))
    for s in (32768, 70000):
        for tol in (0.0, 1e-100):
            U = torch.zeros_like(dev(f))
            hj.solve_vc_2d(dev(a), dev(f), U, hx=0.2, hy=0.3, tile=(16, 16), s=s, rel_tol=tol, max_cycles=3,
                           allow_not_converged=True)
            for b in range(2):
                want, co = orc.vc_solve_2d(a, f[b], np.zeros((5, 6)), 0.2, 0.3, tile=(16, 16), s=s, tol=tol,
                                           max_cycles=3)[:2]
                assert np.array_equal(host(U)[b], want), (s, tol, b)


# solves that would run whole in one workgroup (at most 64 x 64 points, overlaps
# that reach 2 s - 2): by the tile kernels, the single solves' and the batched
# engine's, register body and LDS body, and in one workgroup
@pytest.mark.parametrize("n,tile,s,ov", [((64, 48), (16, 32), 6, (10, 10)), ((64, 48), (16, 16), 4, (6, 6)),
                                         ((64, 48), (64, 32), 8, (14, 14)), ((64, 64), (64, 64), 3, (0, 0)),
                                         ((40, 64), (64, 32), 1, (2, 2)), ((33, 47), (32, 32), 2, (5, 3)),
                                         ((20, 24), (16, 16), 6, (10, 10)), ((1, 1), (16, 16), 1, (0, 0))])
def test_vc_small_solves_by_every_path_match_oracle(orc, n, tile, s, ov):
    nx, ny = n
    hx, hy = 1.0 / (nx + 1), 0.9 / (ny + 1)
    rng = np.random.default_rng(nx + 100 * ny + s)
    a = np.exp(0.5 * rng.standard_normal((ny + 2, nx + 2)))
    f, u0 = rng.standard_normal((3, ny, nx)), rng.standard_normal((3, ny, nx))
    kw = dict(tile=tile, s=s, overlap=ov)
    say(f"vc small by every path {n} {tile} s={s}")
    for tol, cap in ((0.0, 3), (1e-100, 4), (0.3, 10_000)):
        want = [orc.vc_solve_2d(a, f[b], u0[b], hx, hy, tol=tol, max_cycles=cap, **kw) for b in range(3)]
        for nb in (1, 3):
            for path in ({}, {"launch_per_cycle": True}, {"lds_kernel": True}):
                U = dev(u0[:nb])
                infos = hj.solve_vc_2d(dev(a), dev(f[:nb]), U, hx=hx, hy=hy, rel_tol=tol, max_cycles=cap,
                                       allow_not_converged=True, **path, **kw)
                for b, (xo, co, relo, r0o) in enumerate(want[:nb]):
                    assert np.array_equal(host(U)[b], xo), (tol, nb, path, b)
                    assert infos[b].cycles == (co if co >= 0 else cap), (tol, nb, path, b)
                    # sums of at most 4096 squares in another order: 4096 x 2^-53 of each, on either side
                    assert abs(infos[b].r0_norm - r0o) <= 1e-12 * r0o
                    assert abs(infos[b].rel_residual - relo) <= 2e-12 * relo


def test_adjoint_by_every_path_is_the_same():
    rng = np.random.default_rng(9)
    nx, ny = 50, 41
    a = dev(np.exp(0.5 * rng.standard_normal((ny + 2, nx + 2))))
    u, g = dev(rng.standard_normal((3, ny, nx))), dev(rng.standard_normal((3, ny, nx)))
    out = []
    for per_cycle in (False, True):
        lam = torch.zeros_like(g)
        infos, grad = hj.solve_adjoint(a, u, g, lam, 1.0 / 51, tile=(32, 32), s=5, overlap=(8, 9), rel_tol=1e-6,
                                       launch_per_cycle=per_cycle)
        out.append(([i.cycles for i in infos], lam, grad))
    assert out[0][0] == out[1][0]
    assert torch.equal(out[0][1], out[1][1]) and torch.equal(out[0][2], out[1][2])


def _one_column(a, f, u, hy, sweeps):
    """Jacobi sweeps of every 1-wide column of u at once (a shared), in the kernels' order of operations."""
    ihx2, ihy2 = 1.0 / 0.25, 1.0 / (hy * hy)
    c = a[1:-1, 1]
    w, e = 0.5 * (c + a[1:-1, 0]) * ihx2, 0.5 * (c + a[1:-1, 2]) * ihx2
    s, n = 0.5 * (c + a[:-2, 1]) * ihy2, 0.5 * (c + a[2:, 1]) * ihy2
    dinv = 1.0 / ((w + e) + (s + n))
    for _ in range(sweeps):
        p = torch.nn.functional.pad(u, (1, 1))
        u = (f + (s * p[:, :-2] + n * p[:, 2:])) * dinv
    return u


@pytest.mark.parametrize("nb", [65535, 65536, 65537, (1 << 23) + 3])
def test_vc_one_workgroup_solves_of_very_many_right_hand_sides(nb):
    """One launch's worth of right-hand sides, one more, and more than 2^32 threads hold."""
    ny, cycles, s = 16, 2, 3
    gen = torch.Generator(device="cuda").manual_seed(3)
    a = torch.rand(ny + 2, 3, dtype=torch.float64, device="cuda", generator=gen) + 0.5
    f = torch.randn(nb, ny, dtype=torch.float64, device="cuda", generator=gen)
    u = torch.zeros_like(f)
    say(f"vc one workgroup x {nb}")
    pr = hj._vc_problem(a, f.reshape(nb, ny, 1), 0.5, 0.1)
    p = hj.make_params((16, 16), s, rel_tol=0.0, max_cycles=cycles)
    st = hj.load().hj_solve_vc_2d(ctypes.byref(pr), f.data_ptr(), u.data_ptr(), ctypes.byref(p), hj._stream(f), None)
    assert st == hj.HJ_OK, hj.last_error()
    assert torch.equal(u, _one_column(a, f, torch.zeros_like(f), 0.1, s * cycles))


def test_vc_cycles_of_more_threads_than_a_launch_counts():
    """16 x 16 tiles a point apart: with s = 1 a cycle is one classical sweep, whatever their number."""
    n, ov = 5830, 15
    assert hj.axis_tiles(n, 16, ov) ** 2 * 128 > 2 ** 32
    gen = torch.Generator(device="cuda").manual_seed(9)
    a = torch.rand(n + 2, n + 2, dtype=torch.float64, device="cuda", generator=gen) + 0.5
    f = torch.randn(n, n, dtype=torch.float64, device="cuda", generator=gen)
    say("threads, vc")
    for tol in (0.0, 1e-100):
        kw = dict(rel_tol=tol, max_cycles=3, allow_not_converged=True)
        X, Y = torch.zeros_like(f), torch.zeros_like(f)
        hj.solve_vc_2d(a, f, X, 1.0 / (n + 1), tile=(16, 16), s=1, overlap=(ov, ov), **kw)
        hj.solve_vc_2d(a, f, Y, 1.0 / (n + 1), method="global", **kw)
        assert torch.equal(X, Y), tol


# grids and right-hand sides on both sides of where the whole solve in one
# workgroup takes less time than the tile kernels
@pytest.mark.parametrize("n,tile,s", [((3, 64), (16, 64), 8), ((16, 16), (16, 16), 32), ((20, 20), (32, 32), 32),
                                      ((32, 48), (32, 32), 16)])
@pytest.mark.parametrize("nb", [1, 2, 300, 3000])
def test_vc_solves_are_the_same_by_either_way(n, tile, s, nb):
    nx, ny = n
    gen = torch.Generator(device="cuda").manual_seed(nb)
    a = torch.rand(ny + 2, nx + 2, dtype=torch.float64, device="cuda", generator=gen) + 0.5
    f = torch.randn(nb, ny, nx, dtype=torch.float64, device="cuda", generator=gen)
    say(f"vc either way {n} s={s} x {nb}")
    for tol, cap in ((0.0, 3), (1e-3, 40)):
        out = []
        for per_cycle in (False, True):
            U = torch.zeros_like(f)
            infos = hj.solve_vc_2d(a, f, U, 1.0 / (nx + 1), tile=tile, s=s, overlap=tuple(min(2 * s - 2, t - 1) for t in tile),
                                   rel_tol=tol, max_cycles=cap, allow_not_converged=True, launch_per_cycle=per_cycle)
            out.append(([i.cycles for i in infos], U))
        assert out[0][0] == out[1][0] and torch.equal(out[0][1], out[1][1]), tol
