"""Default calls on two streams of one thread, with no wait of the caller's
between them, and of two threads on one stream: no two calls in flight share
their scratch, so the lists of both fields equal the CPU oracle's.  The second field of a pair is the larger one, so the scratch
of the call under way could neither be shared nor outgrown."""
import threading

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


@pytest.mark.parametrize("own_streams", [False, True])
def test_two_threads(own_streams):
    dims = [(24, 20, 16), (64, 50, 41)]
    cases = [_case(d, 3 + i) for i, d in enumerate(dims)]
    torch.cuda.synchronize()
    print("two threads", own_streams, flush=True)
    got, errors = [[], []], []
    start = threading.Barrier(2)

    def work(i):
        try:
            start.wait(30)
            with torch.cuda.stream(torch.cuda.Stream() if own_streams else None):
                for _ in range(20):
                    o, _, lists, _ = dms.gradient_pipeline(cases[i][0])
                    got[i].append((o, lists))
                    got[i].append((o, dms.critical_simplices(cases[i][2], dims[i])[0]))
        except Exception as e:  # raised in the main thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    if errors:
        raise errors[0]
    torch.cuda.synchronize()
    for i in range(2):
        assert len(got[i]) == 40
        for o, lists in got[i]:
            assert (o.cpu().numpy() == cases[i][1]).all()
            _same(lists, cases[i][3])
