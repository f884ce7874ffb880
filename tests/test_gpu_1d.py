"""Grids of one dimension, whose products, energies and gradients run whole in
one workgroup: every length, spin and precision against the oracle at the
tolerances of the other field comparisons (1e-11 FP64, 1e-5 mixed, 1e-10 on
energies).  Length 512 with spin 3 takes more than 64 KB of LDS, as do the x
passes of that length in more dimensions."""
import numpy as np
import pytest

import oracle
from paper_1907_01194_amd import workloads as W
from helpers import oracle_problem, small_spec

pytestmark = pytest.mark.gpu

SIZES = (4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512)


def setup(F, grid, seed):
    spec = small_spec(F, grid, p=0.1, q=0.05)
    prob = oracle_problem(spec)
    u = oracle.retraction.psi(prob, W.noisy_envelope_state(spec, seed, (0.2,) * len(grid)), 1)
    return spec, prob, u, oracle.project(prob, u, W.random_direction(spec, seed + 1))


@pytest.mark.parametrize("F", [1, 2, 3])
@pytest.mark.parametrize("n", SIZES)
def test_product_1d(F, n):
    import torch
    from paper_1907_01194_amd.binding import Problem
    from gpu_util import assert_field, dev, host
    print("1D product", F, n, flush=True)
    spec, prob, u, xi = setup(F, (n,), n)
    ref_e, ref_r = oracle.hvp(prob, u, xi), oracle.rhess(prob, u, xi, sigma=0.2)
    k_or = oracle.inner(xi, ref_r)
    for precision, tol in (("fp64", 1e-11), ("mixed", 1e-5)):
        gp = Problem(spec, precision)
        gp.set_point(dev(u))
        Z = dev(xi, gp.work_dtype)
        assert_field(host(gp.hvp(Z)), ref_e, tol, "hvp")
        assert_field(host(gp.hvp(Z, riemannian=True, sigma=0.2)), ref_r, tol, "rhess")
        HR, kappa = gp.hvp_dot(Z, 0.2)
        assert_field(host(HR), ref_r, tol, "rhess with kappa")
        assert abs(kappa - k_or) <= tol * abs(k_or)
        gp.close()


@pytest.mark.parametrize("F", [2, 3])
@pytest.mark.parametrize("n", SIZES)
def test_energy_and_gradients_1d(F, n):
    import torch
    from paper_1907_01194_amd.binding import Problem
    from gpu_util import assert_field, dev, host
    print("1D energy and gradients", F, n, flush=True)
    spec, prob, u, _ = setup(F, (n,), n + 2)
    E_or = oracle.energy(prob, u)
    gp = Problem(spec, "fp64")
    X = dev(u)
    assert abs(gp.energy(X) - E_or) <= 1e-10 * abs(E_or)
    for riem, ref in ((False, oracle.grad(prob, u)), (True, oracle.rgrad(prob, u)[0])):
        G, E, gn = gp.grad(X, riemannian=riem)
        assert abs(E - E_or) <= 1e-10 * abs(E_or)
        assert_field(host(G), ref, 1e-11, "gradient")
        assert abs(gn - np.linalg.norm(ref)) <= 1e-11 * gn
    gp.close()


@pytest.mark.parametrize("F,grid", [(1, (128,)), (3, (512,)), (3, (512, 6))])
def test_captured_product(F, grid):
    """gpe_hvp only launches, so it can be captured, with a kernel of more than 64 KB
    of LDS too: replays on changed directions, with the handle's own work in
    between, are the eager product's bit for bit."""
    import torch
    from paper_1907_01194_amd.binding import Problem
    from gpu_util import dev
    print("captured product", F, grid, flush=True)
    spec, prob, u, xi = setup(F, grid, 3)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        gp = Problem(spec, "fp64")
        X = dev(u)
        gp.set_point(X)
        Z, H = dev(xi), gp.empty(work=True)
        eager = gp.hvp(Z, riemannian=True, sigma=0.2)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            gp.hvp(Z, riemannian=True, sigma=0.2, out=H)
        for rep in range(4):
            Z.copy_(dev(W.random_direction(spec, 10 + rep)))
            eager = gp.hvp(Z, riemannian=True, sigma=0.2)
            gp.energy(X)
            H.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(H, eager), rep
        del g
        gp.close()
