"""Line transforms of every supported length, as contiguous (x) and strided (y)
lines with tiles that are only partly filled: the Hessian-vector product of a
2D problem against the oracle, FP64 and mixed.  The tolerances are those of the
other field comparisons (1e-11, 1e-5): an error of a transform is a few ulps
times log2 n, about 5e-15 and 1e-6 at n = 512."""
import numpy as np
import pytest

import oracle
from oracle.multigrid import prolong as oracle_prolong
from paper_1907_01194_amd import workloads as W
from helpers import oracle_problem, small_spec

pytestmark = pytest.mark.gpu

SIZES = (4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", SIZES)
def test_every_line_length(n, precision):
    import torch
    from paper_1907_01194_amd.binding import Problem
    from gpu_util import dev, host, assert_field
    tol = 1e-11 if precision == "fp64" else 1e-5
    # 6 and 12 lines per component: no tile of 8, 16 or 64 lines is full; 48: some are
    for F, grid in ((1, (n, 6)), (2, (12, n)), (1, (48, n))):
        print("line length", n, "grid", grid, precision, flush=True)
        spec = small_spec(F, grid)
        prob = oracle_problem(spec)
        u = oracle.retraction.psi(prob, W.noisy_envelope_state(spec, n, (0.2, 0.2)), 1)
        xi = oracle.project(prob, u, W.random_direction(spec, n + 1))
        gp = Problem(spec, precision)
        gp.set_point(dev(u))
        Z = dev(xi, gp.work_dtype)
        assert_field(host(gp.hvp(Z, riemannian=False)), oracle.hvp(prob, u, xi), tol, "hvp")
        HR, kappa = gp.hvp_dot(Z, 0.2)
        ref = oracle.rhess(prob, u, xi, sigma=0.2)
        assert_field(host(HR), ref, tol, "rhess")
        k_or = oracle.inner(xi, ref)
        assert abs(kappa - k_or) <= tol * abs(k_or)
        gp.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("F,grid", [(1, (192, 192)), (3, (192, 96)), (2, (192, 16, 24)), (2, (192, 512)),
                                    (1, (192, 48, 64)), (2, (192, 64, 48)), (1, (192, 48, 48))])
def test_untuned_length_schedules(F, grid, precision):
    """The x pass of length 192 on either side of the lines between its one-row,
    128- and 256-thread schedules (2^17 and 2^19 points), the last workgroup
    partly filled (5 or 3 rows of 3072): the product against the oracle at the
    tolerances above."""
    import torch
    from paper_1907_01194_amd.binding import Problem
    from gpu_util import dev, host, assert_field
    print("schedules", F, grid, precision, flush=True)
    tol = 1e-11 if precision == "fp64" else 1e-5
    spec = small_spec(F, grid)
    prob = oracle_problem(spec)
    u = oracle.retraction.psi(prob, W.noisy_envelope_state(spec, 5, (0.2,) * len(grid)), 1)
    xi = oracle.project(prob, u, W.random_direction(spec, 6))
    gp = Problem(spec, precision)
    gp.set_point(dev(u))
    HR, kappa = gp.hvp_dot(dev(xi, gp.work_dtype), 0.2)
    ref = oracle.rhess(prob, u, xi, sigma=0.2)
    assert_field(host(HR), ref, tol, "rhess")
    k_or = oracle.inner(xi, ref)
    assert abs(kappa - k_or) <= tol * abs(k_or)
    gp.close()


@pytest.mark.parametrize("n", SIZES)
def test_energy_and_gradients_every_line_length(n):
    """The energy (forward transforms and Parseval sums only), the Euclidean and
    the Riemannian gradient with their norms (the latter through the last axis'
    own sums) against the oracle: 1e-10 relative on E, 1e-11 on fields."""
    import torch
    from paper_1907_01194_amd.binding import Problem
    from gpu_util import dev, host, assert_field
    for F, grid in ((1, (n,)), (3, (n, 6)), (2, (12, n)), (1, (6, 8, n)), (1, (8, n, 4))):
        print("energy / gradient, line length", n, "grid", grid, flush=True)
        spec = small_spec(F, grid, p=0.1, q=0.05)
        prob = oracle_problem(spec)
        u = oracle.retraction.psi(prob, W.noisy_envelope_state(spec, n, (0.2,) * len(grid)), 1)
        E_or, G_or = oracle.energy(prob, u), oracle.grad(prob, u)
        gR_or = oracle.rgrad(prob, u)[0]
        gp = Problem(spec, "fp64")
        X = dev(u)
        assert abs(gp.energy(X) - E_or) <= 1e-10 * abs(E_or)
        for riem, ref in ((False, G_or), (True, gR_or)):
            G, E, gn = gp.grad(X, riemannian=riem)
            assert abs(E - E_or) <= 1e-10 * abs(E_or)
            assert_field(host(G), ref, 1e-11, "gradient")
            assert abs(gn - np.linalg.norm(ref)) <= 1e-11 * gn
        gp.close()


@pytest.mark.parametrize("F,grid", [(1, (256, 32, 32)), (2, (96, 64, 48)), (3, (64, 64, 64)), (1, (512, 512)),
                                    (2, (192, 32, 48))])
def test_gradient_dense_rows(F, grid):
    """Grids from 2^18 points on, several x rows a workgroup and a last one that
    is only partly filled (256: 5 rows of 1024; 512: one row): energy and
    Riemannian gradient against the oracle at the tolerances above."""
    import torch
    from paper_1907_01194_amd.binding import Problem
    from gpu_util import dev, host, assert_field
    print("dense rows", F, grid, flush=True)
    spec = small_spec(F, grid, p=0.1, q=0.05)
    prob = oracle_problem(spec)
    u = oracle.retraction.psi(prob, W.noisy_envelope_state(spec, 3, (0.2,) * len(grid)), 1)
    ref, E_or = oracle.rgrad(prob, u)[0], oracle.energy(prob, u)
    gp = Problem(spec, "fp64")
    X = dev(u)
    assert abs(gp.energy(X) - E_or) <= 1e-10 * abs(E_or)
    G, E, gn = gp.grad(X, riemannian=True)
    assert abs(E - E_or) <= 1e-10 * abs(E_or)
    assert_field(host(G), ref, 1e-11, "gradient")
    assert abs(gn - np.linalg.norm(ref)) <= 1e-11 * gn
    gp.close()


@pytest.mark.parametrize("n", SIZES)
def test_equal_axes(n):
    """Axes of the x axis' length, whose sums share the x pass' launch: energy and
    Riemannian gradient of square, of cubic and of mixed grids (y or z alone of
    x's length) against the oracle at the tolerances above."""
    import torch
    from paper_1907_01194_amd.binding import Problem
    from gpu_util import dev, host, assert_field
    grids = [(1, (n, n)), (2, (n, 4, n)), (3, (n, n, 6))] + ([(1, (n, n, n))] if n <= 64 else [])
    for F, grid in grids:
        print("equal axes", F, grid, flush=True)
        spec = small_spec(F, grid, p=0.1, q=0.05)
        prob = oracle_problem(spec)
        u = oracle.retraction.psi(prob, W.noisy_envelope_state(spec, n, (0.2,) * len(grid)), 1)
        ref, E_or = oracle.rgrad(prob, u)[0], oracle.energy(prob, u)
        gp = Problem(spec, "fp64")
        X = dev(u)
        assert abs(gp.energy(X) - E_or) <= 1e-10 * abs(E_or)
        G, E, gn = gp.grad(X, riemannian=True)
        assert abs(E - E_or) <= 1e-10 * abs(E_or)
        assert_field(host(G), ref, 1e-11, "gradient")
        assert abs(gn - np.linalg.norm(ref)) <= 1e-11 * gn
        gp.close()


@pytest.mark.parametrize("n", [s for s in SIZES if 2 * s in SIZES])
def test_prolong_every_line_length(n):
    """Fourier prolongation of every coarse length, as a contiguous and as a
    strided axis with partly filled tiles, against the oracle: 1e-12 on fields
    (one forward and one inverse transform per axis, a few ulps times log2 n)."""
    import torch
    from paper_1907_01194_amd.binding import Problem
    from gpu_util import dev, host, assert_field
    for F, grid in ((2, (n,)), (1, (n, 6)), (3, (4, n)), (1, (6, 4, n))):
        print("prolong, coarse length", n, "grid", grid, flush=True)
        sc, sf = small_spec(F, grid), small_spec(F, tuple(2 * m for m in grid))
        Xc = W.random_direction(sc, n)
        pc, pf = Problem(sc, "fp64"), Problem(sf, "fp64")
        assert_field(host(pc.prolong(dev(Xc), pf)), oracle_prolong(oracle_problem(sc), Xc), 1e-12, "prolong")
        pc.close()
        pf.close()
