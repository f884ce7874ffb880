"""Rules that choose between launches by the size of the grid: which calls take
which path, and that every path gives the oracle's results."""
import numpy as np
import pytest

import oracle
from paper_1907_01194_amd import workloads as W
from helpers import oracle_problem, small_spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,grid,local", [(1, (16, 16), True), (3, (512, 384), True), (3, (64, 64, 48), True),
                                          (2, (96, 48, 48), True), (3, (64, 64, 64), True), (2, (64, 64, 64), True),
                                          (1, (128, 64, 48), False)])
def test_cg_step_launches(F, grid, local):
    """A CG iteration on a grid of up to 2^18 points has one finalize (the
    curvature's), its closing step applying the residual and cap tests itself;
    beyond, two.  Counted as the difference between a run with 2 iterations
    queued and one with 6 (no line search follows, and the shift keeps the
    Hessian positive: a curvature stop takes one more inner product)."""
    import torch
    from paper_1907_01194_amd.binding import Problem
    from gpu_util import dev
    print("CG launches", F, grid, flush=True)
    spec = small_spec(F, grid)
    u = W.noisy_envelope_state(spec, 1, (0.2,) * len(grid))
    gp = Problem(spec, "mixed")
    n = {}
    for cap in (2, 3):
        gp.timing(True)
        gp.newton_solve(dev(u), check=False, rgbb_maxit=0, maxit=1, ls_max=0, cg_maxit=cap, cg_T=1e-12,
                        cg_per_digit=0.0, sigma_hat0=100.0, tol=1e-14)
        n[cap] = gp.timing_read()
    gp.close()
    assert n[3]["hvp_xpass"][0] - n[2]["hvp_xpass"][0] == 4
    assert n[3]["finalize"][0] - n[2]["finalize"][0] == (4 if local else 8)


@pytest.mark.parametrize("F,grid,count,timed", [(1, (64, 16), 3, False), (2, (64, 64), 3, False),
                                                (3, (96, 16), 3, False), (1, (128, 128), 3, False),
                                                (2, (192, 16), 3, False), (3, (256, 512), 3, False),
                                                (1, (192, 32, 24), 3, True), (2, (64, 64, 64), 3, True),
                                                (1, (192, 48, 64), 3, True), (1, (48, 48), 1, False),
                                                (1, (512, 512), 1, False)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_schedule_chosen(F, grid, count, timed, precision):
    """Every x length from 64 to 256 has three schedules: grids of up to 2^17
    points take the last untimed, larger ones the fastest of the three, whose
    times are on record.  The other lengths have one."""
    import torch
    from paper_1907_01194_amd.binding import Problem
    print("schedule", F, grid, precision, flush=True)
    gp = Problem(small_spec(F, grid), precision)
    v, us = gp.schedule()
    assert gp.schedule_count() == count
    if timed:
        assert all(t > 0 for t in us) and us[v] == min(us)
    else:
        assert us == [0, 0, 0] and v == (2 if count == 3 else 1)
    gp.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("F,grid", [(F, (n, 6)) for n in (64, 96, 128, 192, 256) for F in (1, 2, 3)] +
                         [(1, (64, 96, 96)), (2, (64, 128, 64)), (1, (96, 96, 64)), (1, (128, 96, 48)),
                          (1, (192, 48, 64)), (3, (192, 64, 48)), (1, (256, 48, 48)), (2, (256, 64, 32))])
def test_every_schedule(F, grid, precision):
    """The product with each schedule forced, on grids on either side of the line
    (2^19 points) between the last one's two forms, the last workgroup partly
    filled wherever the rows do not divide: against the oracle at the
    tolerances of the other field comparisons."""
    import torch
    from paper_1907_01194_amd.binding import Problem
    from gpu_util import assert_field, dev, host
    print("every schedule", F, grid, precision, flush=True)
    tol = 1e-11 if precision == "fp64" else 1e-5
    spec = small_spec(F, grid)
    prob = oracle_problem(spec)
    u = oracle.retraction.psi(prob, W.noisy_envelope_state(spec, 7, (0.2,) * len(grid)), 1)
    xi = oracle.project(prob, u, W.random_direction(spec, 8))
    ref = oracle.rhess(prob, u, xi, sigma=0.2)
    k_or = oracle.inner(xi, ref)
    gp = Problem(spec, precision)
    gp.set_point(dev(u))
    Z = dev(xi, gp.work_dtype)
    assert gp.schedule_count() == 3
    for v in range(3):
        gp.set_schedule(v)
        assert gp.schedule()[0] == v
        HR, kappa = gp.hvp_dot(Z, 0.2)
        assert_field(host(HR), ref, tol, "rhess, schedule %d" % v)
        assert abs(kappa - k_or) <= tol * abs(k_or)
    gp.close()
