"""Fields with short sides: so many of their vertices lie on the boundary, where
no lower-star table applies, that the queue of such vertices fills up.  Tiles
solve the rest themselves in launches of more than 1024 tiles and list it in
smaller ones.  Records and the critical mask must equal the CPU
oracle's exactly, from ranks and from values, and in batches of each tile
shape."""
import numpy as np
import pytest

import oracle
import paper_2505_21266_amd as dms
from batch_cache import pin_variant

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [
    (20, 30, 300),   # 600 tiles: listed
    (20, 30, 700),   # 1400: boundary columns and rows, the queue fills late
    (12, 16, 1024),  # one tile a plane, a third of it general; the most tiles that list
    (12, 16, 1025),  # one more
    (3, 85, 300),    # five full tiles of 48 and one of 15 a plane, all but a column general
    (255, 2, 260),   # four tiles a plane, every vertex general, none of them dense
]


def _field(dims, kind, seed=0):
    nx, ny, nz = dims
    if kind == "ties":
        return np.random.default_rng(seed).integers(0, 3, (nz, ny, nx)).astype(np.float32)
    x, y, z = (np.linspace(0.3, 0.3 + a + 0.1 * seed, n) for a, n in zip((3.0, 4.0, 9.0), dims))
    return (np.sin(z)[:, None, None] + np.cos(y)[None, :, None] + np.sin(x)[None, None, :]).astype(np.float32)


def _mask_bits(mask, n):
    return np.unpackbits(mask.cpu().numpy().view(np.uint8), bitorder="little")[:n].astype(bool)


def _flagged(rec, dims, n):
    lists, _ = oracle.critical_simplices(rec, dims)
    flagged = np.zeros(n, bool)
    for codes in lists:
        flagged[codes >> 8] = True
    return flagged


@pytest.mark.parametrize("dims", SHAPES)
@pytest.mark.parametrize("kind", ["smooth", "ties"])
def test_full_queue(dims, kind):
    v = _field(dims, kind)
    o = oracle.order(v)
    want, _, _ = oracle.lower_stars(o, dims)
    n = o.size
    flagged = _flagged(want, dims, n)
    og = torch.from_numpy(o).cuda().reshape(dims[::-1])
    for form in ("ranks", "f32", "f64"):
        print("full queue", dims, kind, form, flush=True)
        mask = dms.critical_mask(n, og.device)
        if form == "ranks":
            got = dms.discrete_gradient(og, mask=mask)
        else:
            vg = torch.from_numpy(v.astype(np.float32 if form == "f32" else np.float64)).cuda()
            got = dms.discrete_gradient_values(vg, mask=mask)
        assert (got.cpu().numpy().view(np.uint32) == want).all(), form
        assert (_mask_bits(mask, n) == flagged).all(), form


@pytest.mark.parametrize("variant", [0, 1, 2])
def test_full_queue_batch(variant, tmp_path):
    sides = [(12 + f % 5, 9 + f % 7, 10 + f % 3) for f in range(120)]
    fields = [_field(s, "ties" if f % 4 == 0 else "smooth", f) for f, s in enumerate(sides)]
    vals = torch.from_numpy(np.concatenate([f.reshape(-1) for f in fields])).cuda()
    b = dms.Batch(sides, cache=pin_variant(tmp_path / "tune", sides, variant))
    print("full queue batch", variant, flush=True)
    order, rec, lists, counts, offsets = b.run(vals)
    assert b.variant == variant
    rec, offsets = rec.cpu().numpy().view(np.uint32), offsets.cpu().numpy()
    lists = [t.cpu().numpy() for t in lists]
    at = 0
    for f, (s, v) in enumerate(zip(sides, fields)):
        n = v.size
        want, _, _ = oracle.lower_stars(oracle.order(v), s)
        assert (rec[at:at + n] == want).all(), f
        at += n
        crit, _ = oracle.critical_simplices(want, s)
        for d in range(4):
            assert (lists[d][offsets[d, f]:offsets[d, f + 1]] == crit[d]).all(), (f, d)
