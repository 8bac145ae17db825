"""A NaN in the field, through the calls that look for it only after the gradient
and the count: the pipeline with and without capacities, and both persistence
functions.  The fields lie below and above the short order's 2^21 values."""
import numpy as np
import pytest

import paper_2505_21266_amd as dms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape", [(5, 6, 7), (30, 40, 50), (129, 128, 130)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("at", [0, -1])
def test_pipeline_nan(shape, dtype, at):
    v = torch.rand(shape, dtype=dtype, device="cuda")
    v.view(-1)[at] = float("nan")
    print("pipeline nan", shape, dtype, at, flush=True)
    with pytest.raises(ValueError, match="NaN"):
        dms.gradient_pipeline(v)
    with pytest.raises(ValueError, match="NaN"):
        dms.gradient_pipeline(v, cap=[v.numel()] * 4)
    # lists without room do not hide it
    with pytest.raises(ValueError, match="NaN"):
        dms.gradient_pipeline(v, cap=[0, 0, 0, 0])
    for f in (dms.PersistenceD0, dms.PersistenceD2):
        with pytest.raises(ValueError, match="NaN"):
            f.apply(v.clone().requires_grad_())


def test_pipeline_infinities():
    v = torch.rand((20, 21, 22), device="cuda")
    v[3, 4, 5], v[6, 7, 8] = float("inf"), float("-inf")
    w = v.clone()
    w[3, 4, 5], w[6, 7, 8] = 2.0, -1.0
    a, b = dms.gradient_pipeline(v), dms.gradient_pipeline(w)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    assert all(torch.equal(x, y) for x, y in zip(a[2], b[2]))
