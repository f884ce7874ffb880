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
