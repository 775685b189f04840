"""The native call module on a host without a GPU: what it does not take is left to the
Python code, which names what is wrong."""
import numpy as np
import pytest

pytest.importorskip("torch")


def test_native_calls_leave_odd_arguments_to_python():
    # nothing is launched: wrong counts, wrong types, host tensors
    import torch

    import paper_1911_08020_amd as darb
    plan = darb.Plan(8, 64, np.full(8, 0.1), 0.1)
    t = torch.zeros(64)
    for fn, n in (("spmv", 6), ("spmv_packed", 6), ("spmv_i8", 8), ("spmm", 6),
                  ("spmm_packed", 6), ("spmm_i8", 8), ("encode", 5)):
        f = getattr(darb._native, fn)
        assert f() is None and f(*range(n)) is None
        assert f(plan._ref, *[t] * (n - 2), None) is None
    with pytest.raises(ValueError):
        plan.spmv(t, t.to(torch.uint8), t)
