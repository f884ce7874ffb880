"""Batch.hvp's marshalling: the directions may be any iterable, one that can be
gone through only once included, and results the call allocates have each
problem's shape and type.  The library is replaced by a recorder, so this runs
without a GPU."""
import ctypes
import itertools

import pytest
import torch

from paper_1907_01194_amd import binding


class _Problem:
    def __init__(self, shape):
        self.shape = shape
        self.work_dtype = torch.complex64

    def empty(self, work=False):
        return torch.empty(self.shape, dtype=self.work_dtype if work else torch.complex128)

    def _w(self, Z):
        assert tuple(Z.shape) == self.shape and Z.dtype == self.work_dtype
        return ctypes.c_void_p(Z.data_ptr())


class _Lib:
    def gpe_batch_hvp(self, b, zp, hp, riem, sg, kap):
        self.z, self.h = list(zp), list(hp)
        return 0 if all(self.z) and all(self.h) else 1

    def gpe_batch_last_error(self, b):
        return b"NULL field"


@pytest.mark.parametrize("wrap", [list, tuple, iter, lambda zs: (Z for Z in zs), lambda zs: map(lambda Z: Z, zs),
                                  lambda zs: itertools.chain(zs, itertools.repeat(None))])
def test_batch_hvp_takes_any_iterable(wrap, monkeypatch):
    rec = _Lib()
    monkeypatch.setattr(binding, "lib", lambda: rec)
    b = binding.Batch.__new__(binding.Batch)
    b.torch, b.b = torch, None
    b.problems = [_Problem((3, 16, 32)), _Problem((3, 64, 16))]
    Zs = [p.empty(work=True) for p in b.problems]
    outs, kap = b.hvp(wrap(Zs), kappa=False)
    assert kap is None
    assert rec.z == [Z.data_ptr() for Z in Zs]
    assert [tuple(H.shape) for H in outs] == [p.shape for p in b.problems]
    assert all(H.dtype == torch.complex64 for H in outs)
    assert rec.h == [H.data_ptr() for H in outs]
