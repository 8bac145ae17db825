"""Host copies of GPU tensors: through pinned memory up to a bound, and beyond
it through memory that is not kept for the process."""
import numpy as np
import pytest

import paper_2505_21266_amd as dms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("over", [-16, 0, 16])
def test_fetch_bound(over, monkeypatch):
    monkeypatch.setattr(dms, "_PINNED_MOST", 1 << 20)
    a = torch.arange(((1 << 20) + over) // 8 - 4, dtype=torch.int64, device="cuda")
    b = torch.arange(5, dtype=torch.int32, device="cuda")  # 20 bytes, 32 with the padding
    none = torch.zeros(0, dtype=torch.int64, device="cuda")
    got = dms._fetch(a, none, b)
    assert [g.dtype for g in got] == [np.int64, np.int64, np.int32]
    assert (got[0] == np.arange(a.numel())).all() and got[1].size == 0 and (got[2] == np.arange(5)).all()
    assert torch.from_numpy(got[0]).is_pinned() == (over <= 0)
