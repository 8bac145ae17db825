"""Long orders (the radix passes over whole and partial tiles, the (id,
position) pairs, both levels of the inversion) against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_21266_amd as dms

pytestmark = pytest.mark.gpu

SHORT = 1 << 21  # longer arrays take the passes tested here
FINE = 1 << 22  # from here on the inversion has its second level


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [SHORT + 1, SHORT + 4096, SHORT + 8191, SHORT + 8192, FINE, FINE + 1, FINE + 8192])
@pytest.mark.parametrize("kind", ["noise", "few", "constant"])
def test_long_order(n, dtype, kind):
    r = np.random.default_rng(n)
    if kind == "noise":
        v = r.standard_normal(n).astype(dtype)
    elif kind == "few":
        v = r.integers(-3, 4, n).astype(dtype)
    else:
        v = np.full(n, -0.5, dtype)
    want = oracle.order(v)
    # aligned, and aligned to one value only
    for skip in (0, 1):
        x = torch.empty(n + skip, dtype=torch.from_numpy(v).dtype, device="cuda")[skip:]
        x.copy_(torch.from_numpy(v))
        got = dms.order(x)
        assert np.array_equal(got.cpu().numpy(), want), (n, skip)
