"""The binding asks for the workspace size once per (n, clusters): by their
values, also where the caller hands over an object whose value changes."""
import ctypes as C

import numpy as np
import pytest


@pytest.mark.parametrize("make", [lambda: np.array(1000), lambda: __import__("torch").tensor(1000)],
                         ids=["numpy", "torch"])
def test_counts_are_compared_by_value(monkeypatch, make):
    from paper_2602_13385_amd import scf

    asked = []

    class Lib:
        def scf_workspace_size(self, handle, n, nclusters, out):
            asked.append((n, nclusters))
            C.cast(out, C.POINTER(C.c_size_t))[0] = 256 * n
            return 0

    monkeypatch.setattr(scf, "lib", Lib)
    plan = object.__new__(scf.Plan)
    plan._h, plan._ws, plan._need = None, None, (None, 0)
    n = make()
    assert plan.workspace(n, device="cpu").numel() == 256_000
    assert plan.workspace(n, device="cpu").numel() == 256_000
    n += 1000  # in place: the same object
    assert plan.workspace(n, device="cpu").numel() == 512_000
    assert plan.workspace(2000, device="cpu").numel() == 512_000
    assert asked == [(1000, 1), (2000, 1)]
