"""The gradient without a workspace: tiles with few vertices that no lower-star
table covers solve them themselves, tiles with many mark their first record for
the kernel behind.  That record may be a table's, a general vertex's or the
tile's only one of its kind.  Records and the critical mask must equal the CPU
oracle's exactly, from ranks and from values, also in a box within the grid."""
import numpy as np
import pytest

import oracle
import paper_2505_21266_amd as dms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _mixed(dims, seed):
    """A ramp (its inner vertices all have a table entry) with noise in some
    tiles: everywhere but in the tile's first row, in its first row only, or all over."""
    nx, ny, nz = dims
    rng = np.random.default_rng(seed)
    z, y, x = np.meshgrid(*(np.arange(n, dtype=np.float64) for n in (nz, ny, nx)), indexing="ij")
    v = (x * 1.0 + y * 1.3 + z * 1.7) * 1e-3
    for t in range(nz):
        how = t % 5
        r = rng.random((ny, nx))
        rows = np.arange(ny) % 16
        if how == 1:
            v[t][rows > 1] += r[rows > 1]
        elif how == 2:
            v[t][rows == 0] += r[rows == 0]
        elif how == 3:
            v[t] += r
    return v.astype(np.float32)


def _check(got, mask, want, n, dims, what):
    assert (got.cpu().numpy().view(np.uint32) == want).all(), what
    lists, _ = oracle.critical_simplices(want, dims)
    flagged = np.zeros(n, bool)
    for codes in lists:
        flagged[codes >> 8] = True
    bits = np.unpackbits(mask.cpu().numpy().view(np.uint8), bitorder="little")[:n].astype(bool)
    assert (bits == flagged).all(), what


# tiles of 64 x 16 x 1; launches of up to 2048 tiles mark none
@pytest.mark.parametrize("dims", [(64, 16, 300), (64, 16, 2048), (64, 16, 2049), (67, 35, 400), (130, 50, 190)])
def test_no_queue(dims):
    v = _mixed(dims, 5)
    o = oracle.order(v)
    want, _, _ = oracle.lower_stars(o, dims)
    og = torch.from_numpy(o).cuda().reshape(dims[::-1])
    for form in ("ranks", "f32", "f64"):
        print("no queue", dims, form, flush=True)
        mask = dms.critical_mask(o.size, og.device)
        if form == "ranks":
            got = dms.discrete_gradient(og, queue=False, mask=mask)
        else:
            vg = torch.from_numpy(v.astype(np.float32 if form == "f32" else np.float64)).cuda()
            got = dms.discrete_gradient_values(vg, queue=False, mask=mask)
        _check(got, mask, want, o.size, dims, form)


def test_no_queue_box():
    dims, lo, hi = (90, 40, 400), (3, 2, 1), (77, 39, 398)
    v = _mixed(dims, 6)
    o = oracle.order(v)
    want, _, _ = oracle.lower_stars(o, dims, lo, hi)
    og = torch.from_numpy(o).cuda().reshape(dims[::-1])
    print("no queue box", flush=True)
    a = dms.discrete_gradient(og, lo, hi, queue=False)
    assert (a.cpu().numpy().view(np.uint32) == want).all()
    assert torch.equal(a, dms.discrete_gradient(og, lo, hi))


def test_no_queue_many_tiles():
    # 400,000 tiles of two vertices: each block asks for its tiles twice; equal to the queue's records
    vals = torch.rand((400000, 1, 2), device="cuda")
    og = dms.order(vals)
    print("no queue many tiles", flush=True)
    assert torch.equal(dms.discrete_gradient(og, queue=False), dms.discrete_gradient(og))
    # the same number of tiles, 16 of 400 dense
    wide = torch.linspace(0, 1, 400000, device="cuda")[:, None, None] + torch.zeros((400000, 16, 17), device="cuda")
    noise = torch.rand((16000, 16, 17), device="cuda")
    wide[torch.arange(400000, device="cuda") % 400 < 16] += noise[:16000]
    og = dms.order(wide)
    assert torch.equal(dms.discrete_gradient(og, queue=False), dms.discrete_gradient(og))
