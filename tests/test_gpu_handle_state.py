"""What a call leaves behind and what it refuses: checks of results that the
caller does not ask for, and the state of a handle after a call that failed."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_1907_01194_amd import workloads as W
from helpers import oracle_problem, small_spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,grid", [(1, (16,)), (3, (512,)), (2, (16, 12)), (1, (8, 6, 8))])
def test_gradient_norm_checked_unasked(F, grid):
    """A Riemannian gradient whose norm overflows is GPE_ENUMERIC, whether or not
    the caller takes the norm (NULL): one huge value of V leaves E, <X, G> and
    ||X||^2 finite (about 1e198) and ||G||^2 infinite."""
    import torch
    from paper_1907_01194_amd import binding as B
    from gpu_util import dev
    print("gradient norm", F, grid, flush=True)
    spec = small_spec(F, grid)
    X = dev(oracle.retraction.psi(oracle_problem(spec), W.noisy_envelope_state(spec, 1, (0.2,) * len(grid)), 1))
    spec.V = spec.V.copy()
    spec.V.flat[spec.V.size // 2] = 1e200
    gp = B.Problem(spec, "fp64")
    G = gp.empty()
    E, gn = ctypes.c_double(), ctypes.c_double()
    for norm in (None, ctypes.byref(gn)):
        st = B.lib().gpe_grad(gp.h, ctypes.c_void_p(X.data_ptr()), ctypes.c_void_p(G.data_ptr()), 1, ctypes.byref(E),
                              norm)
        assert st == 4, (st, norm)
    assert np.isfinite(E.value)
    gp.close()
