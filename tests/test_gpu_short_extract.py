"""The extraction of short boxes (up to 4096 tiles of 1024 records, filled a
group of 128 records at a time): sizes at the edges of groups and tiles and on
both sides of the limit, with and without the mask, truncated lists, and the
same in a batch.  Lists and counts must equal the CPU oracle's exactly."""
import numpy as np
import pytest

import oracle
import paper_2505_21266_amd as dms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(1, 1, 1), (127, 1, 1), (128, 1, 1), (129, 1, 1), (1, 1023, 1), (32, 32, 1), (1, 1, 1025), (33, 31, 9),
          (128, 128, 256), (128, 128, 257)]


def _records(dims, seed):
    nx, ny, nz = dims
    v = np.random.default_rng(seed).random((nz, ny, nx), dtype=np.float32)
    og = dms.order(torch.from_numpy(v).cuda())
    mask = dms.critical_mask(og.numel(), og.device)
    rec = dms.discrete_gradient(og, mask=mask)
    want, _ = oracle.critical_simplices(rec.cpu().numpy().view(np.uint32), dims)
    return v, rec, mask, want


@pytest.mark.parametrize("dims", SHAPES)
def test_short_lists(dims):
    _, rec, mask, want = _records(dims, sum(dims))
    print("short lists", dims, flush=True)
    for m in (mask, None):
        lists, counts = dms.critical_simplices(rec, dims, mask=m)
        assert counts.cpu().tolist() == [len(w) for w in want]
        for d in range(4):
            assert (lists[d].cpu().numpy() == want[d]).all(), (d, m is None)
        # lists with room for half: the first cells, the exact counts and the flag
        cap = [len(w) // 2 for w in want]
        flags = dms.new_flags(rec.device)
        lists, counts = dms.critical_simplices(rec, dims, cap=cap, flags=flags, mask=m)
        assert counts.cpu().tolist() == [len(w) for w in want]
        assert int(flags.item()) == dms.FLAG_CAPACITY
        for d in range(4):
            assert (lists[d].cpu().numpy() == want[d][:cap[d]]).all(), (d, m is None)


@pytest.mark.parametrize("sides", [[(1, 1, 1), (127, 1, 1), (1, 128, 1), (3, 3, 3)], [(16, 16, 4)] * 40,
                                   [(128, 128, 255), (128, 127, 1), (128, 1, 1)],
                                   [(128, 128, 255), (128, 128, 1), (2, 1, 1)]])
def test_short_batch_lists(sides):
    rng = np.random.default_rng(len(sides))
    fields = [rng.random((nz, ny, nx), dtype=np.float32) for nx, ny, nz in sides]
    vals = torch.from_numpy(np.concatenate([f.reshape(-1) for f in fields])).cuda()
    print("short batch lists", len(sides), vals.numel(), flush=True)
    _, rec, lists, counts, offsets = dms.Batch(sides).run(vals)
    rec, offsets = rec.cpu().numpy().view(np.uint32), offsets.cpu().numpy()
    at = 0
    for f, (nx, ny, nz) in enumerate(sides):
        n = nx * ny * nz
        want, _ = oracle.critical_simplices(rec[at:at + n], (nx, ny, nz))
        at += n
        for d in range(4):
            lo, hi = offsets[d, f], offsets[d, f + 1]
            assert hi - lo == len(want[d]) == int(counts[f, d])
            assert (lists[d][lo:hi].cpu().numpy() == want[d]).all()
