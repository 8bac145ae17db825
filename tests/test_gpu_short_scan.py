"""Extraction of short boxes at the edges of the one-block scan's rows (1024
tile counts each, four a tile), of smooth fields, most of whose groups of 128
records hold no critical cell and are not read, and of noise.  Lists and counts
must equal the CPU oracle's exactly."""
import numpy as np
import pytest

import oracle
import paper_2505_21266_amd as dms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _field(dims, kind):
    nx, ny, nz = dims
    if kind == "noise":
        return np.random.default_rng(nz).random((nz, ny, nx), dtype=np.float32)
    x, y, z = (np.linspace(0.0, a, n) for a, n in zip((5.0, 4.0, 0.05 * nz), dims))
    return (np.sin(z)[:, None, None] + np.cos(y)[None, :, None] + np.sin(x)[None, None, :]).astype(np.float32)


@pytest.mark.parametrize("tiles", [255, 256, 257, 1023, 1024, 4095])
@pytest.mark.parametrize("kind", ["smooth", "noise"])
def test_scan_rows(tiles, kind):
    dims = (32, 32, tiles)
    og = dms.order(torch.from_numpy(_field(dims, kind)).cuda())
    mask = dms.critical_mask(og.numel(), og.device)
    rec = dms.discrete_gradient(og, mask=mask)
    want, _ = oracle.critical_simplices(rec.cpu().numpy().view(np.uint32), dims)
    print("scan rows", tiles, kind, [len(w) for w in want], flush=True)
    for m in (mask, None):
        lists, counts = dms.critical_simplices(rec, dims, mask=m)
        assert counts.cpu().tolist() == [len(w) for w in want]
        for d in range(4):
            assert (lists[d].cpu().numpy() == want[d]).all(), (d, m is None)


def test_scan_rows_batch():
    # 513 fields of 500 to 512 vertices: fields start and end inside groups
    sides = [(8, 8, 8) if f % 3 else (10, 10, 5) for f in range(513)]
    rng = np.random.default_rng(7)
    fields = [rng.random((nz, ny, nx), dtype=np.float32) if f % 2 else
              np.arange(nx * ny * nz, dtype=np.float32).reshape(nz, ny, nx) for f, (nx, ny, nz) in enumerate(sides)]
    vals = torch.from_numpy(np.concatenate([f.reshape(-1) for f in fields])).cuda()
    print("scan rows batch", vals.numel(), flush=True)
    _, rec, lists, counts, offsets = dms.Batch(sides).run(vals)
    rec, offsets, counts = rec.cpu().numpy().view(np.uint32), offsets.cpu().numpy(), counts.cpu().numpy()
    lists = [t.cpu().numpy() for t in lists]
    at = 0
    for f, (nx, ny, nz) in enumerate(sides):
        n = nx * ny * nz
        want, _ = oracle.critical_simplices(rec[at:at + n], (nx, ny, nz))
        at += n
        for d in range(4):
            lo, hi = offsets[d, f], offsets[d, f + 1]
            assert hi - lo == len(want[d]) == counts[f, d]
            assert (lists[d][lo:hi] == want[d]).all()
