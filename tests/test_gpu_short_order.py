"""The order of short inputs: one block for all passes, then tiles of 2048,
4096 and 8192 keys whose scatter blocks sum the digit counts themselves.  The
sizes are the edges between those routes and of their tiles; orders must equal
the CPU oracle's exactly."""
import numpy as np
import pytest

import oracle
import paper_2505_21266_amd as dms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [1, 2, 63, 1025, 8192, 8193, 10240, 10241, (1 << 19) - 1, 1 << 19, (1 << 19) + 1, 1 << 20, (1 << 20) + 1,
         (1 << 21) - 4097, 1 << 21, (1 << 21) + 1]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind", ["noise", "ties"])
def test_short_order(n, dtype, kind):
    rng = np.random.default_rng(n)
    # negative values, both zeros and repeated values among the keys
    v = rng.standard_normal(n).astype(dtype) if kind == "noise" else rng.integers(-2, 3, n).astype(dtype) * dtype(0.5)
    if n > 60:
        v[17], v[58] = -0.0, 0.0
    print("short order", n, np.dtype(dtype).name, kind, flush=True)
    got = dms.order(torch.from_numpy(v).cuda()).cpu().numpy()
    assert (got == oracle.order(v)).all()


@pytest.mark.parametrize("n,at", [(5, 0), (8192, 8191), (8193, 8192), (600000, 599999), (2000000, 4096)])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_short_order_nan_flag(n, at, dtype):
    v = np.random.default_rng(n).random(n).astype(dtype)
    v[at] = np.nan
    with pytest.raises(ValueError):
        dms.order(torch.from_numpy(v).cuda())


@pytest.mark.parametrize("sides", [[(3, 2, 1)], [(20, 19, 21), (1, 1, 7), (2, 3, 4)],
                                   [(40, 41, 42), (5, 60, 7), (64, 64, 65)],
                                   [(7, 6, 5)] * 300, [(128, 64, 64), (129, 65, 66), (3, 3, 3)]])
def test_short_batch_order(sides):
    rng = np.random.default_rng(len(sides))
    fields = [rng.standard_normal((nz, ny, nx)).astype(np.float32) for nx, ny, nz in sides]
    vals = torch.from_numpy(np.concatenate([f.reshape(-1) for f in fields])).cuda()
    print("short batch order", len(sides), vals.numel(), flush=True)
    order = dms.Batch(sides).run(vals)[0].cpu().numpy()
    want = np.concatenate([oracle.order(f).reshape(-1) for f in fields])
    assert (order == want).all()
