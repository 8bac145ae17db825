"""Default calls on two streams of one thread, with no wait of the caller's
between them: each call's scratch is its own, so the lists of both fields equal
the CPU oracle's.  The second field of a pair is the larger one, so the scratch
of the call under way could neither be shared nor outgrown."""
import numpy as np
import pytest

import oracle
import paper_2505_21266_amd as dms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _case(dims, seed):
    nx, ny, nz = dims
    v = np.random.default_rng(seed).random((nz, ny, nx), dtype=np.float32)
    o = oracle.order(v)
    rec, _, _ = oracle.lower_stars(o, dims)
    lists, _ = oracle.critical_simplices(rec, dims)
    return torch.from_numpy(v).cuda(), o, torch.from_numpy(rec.view(np.int32).copy()).cuda(), lists


def _same(lists, want):
    for d in range(4):
        assert (lists[d].cpu().numpy() == want[d]).all(), d


# short boxes beside each other, and beside one past the short forms' limits
@pytest.mark.parametrize("small,large", [((24, 20, 16), (64, 50, 41)), ((64, 64, 64), (161, 163, 165))])
def test_two_streams(small, large):
    cases = [_case(small, 1), _case(large, 2)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    masks = []
    for (nx, ny, nz), (v, o, _, _) in zip((small, large), cases):
        m = dms.critical_mask(nx * ny * nz, v.device)
        dms.discrete_gradient(torch.from_numpy(o).cuda().reshape(nz, ny, nx), mask=m)
        masks.append(m)
    torch.cuda.synchronize()
    for form in ("mask", "nomask", "pipeline"):
        print("two streams", small, large, form, flush=True)
        got = []
        for _ in range(6):
            for s, dims, (v, _, rec, _), m in zip(streams, (small, large), cases, masks):
                with torch.cuda.stream(s):
                    if form == "pipeline":
                        got.append(dms.gradient_pipeline(v)[2])
                    else:
                        got.append(dms.critical_simplices(rec, dims, mask=m if form == "mask" else None)[0])
        torch.cuda.synchronize()
        for i, lists in enumerate(got):
            _same(lists, cases[i % 2][3])


def test_two_streams_order():
    vals = [torch.rand(n, device="cuda") for n in (300000, 2500000)]
    want = [oracle.order(v.cpu().numpy()) for v in vals]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    got = []
    print("two streams order", flush=True)
    for _ in range(6):
        for s, v in zip(streams, vals):
            with torch.cuda.stream(s):
                got.append(dms.order(v, flags=dms.new_flags(v.device), check=False))
    torch.cuda.synchronize()
    for i, o in enumerate(got):
        assert (o.cpu().numpy() == want[i % 2]).all(), i
