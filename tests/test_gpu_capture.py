"""A step recorded into a torch graph (order, gradient, extraction with given
capacities, nothing that waits): replays on new values, with eager calls and
waits between them, equal the CPU oracle.  The workspaces that the calls take
for themselves come from the graph's own memory."""
import functools

import numpy as np
import pytest

import oracle
import paper_2505_21266_amd as dms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@functools.lru_cache(maxsize=None)
def _case(dims, seed):
    nx, ny, nz = dims
    f = np.random.default_rng(seed).random((nz, ny, nx), dtype=np.float32)
    o = oracle.order(f)
    rec, _, _ = oracle.lower_stars(o, dims)
    return f, o, rec, oracle.critical_simplices(rec, dims)[0]


@pytest.mark.parametrize("dims", [(24, 20, 16), (70, 50, 90), (140, 130, 140)])
@pytest.mark.parametrize("queue", [True, False])
def test_captured_step(dims, queue):
    nx, ny, nz = dims
    n = nx * ny * nz
    x = torch.rand((nz, ny, nx), device="cuda")
    mask, flags = dms.critical_mask(n, x.device), dms.new_flags(x.device)
    cap = [n] * 4

    def step():
        o = dms.order(x, flags=flags, check=False)
        rec = dms.discrete_gradient(o, queue=queue, mask=mask)
        lists, counts = dms.critical_simplices(rec, dims, cap=cap, flags=flags, mask=mask)
        return o, rec, lists, counts

    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        step()
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    print("captured step", dims, queue, flush=True)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        o, rec, lists, counts = step()
    for seed in (1, 2, 1):
        f, want_o, want, crit = _case(dims, seed)
        x.copy_(torch.from_numpy(f))
        graph.replay()
        torch.cuda.synchronize()
        assert (o.cpu().numpy() == want_o).all()
        assert (rec.cpu().numpy().view(np.uint32) == want).all()
        assert counts.cpu().tolist() == [len(c) for c in crit] and int(flags.item()) == 0
        for d in range(4):
            assert (lists[d][:len(crit[d])].cpu().numpy() == crit[d]).all(), d
        # eager work of the same kind in between
        e = dms.gradient_pipeline(x)
        assert torch.equal(e[0], o) and torch.equal(e[1], rec)
