"""Ranked integer keys: the backward's contributions over vertex counts that
need two to five radix passes, below and above the short sorts' limit, and
filtration keys of cells given in any order, repeated, and named from a vertex
that is not their highest."""
import numpy as np
import pytest

import paper_2505_21266_amd as dms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("npairs", [3, 5000, 300000, 1100000])
@pytest.mark.parametrize("n", [200, 256, 65535, 65536, (1 << 24) + 3])
def test_backward_pass_counts(npairs, n):
    rng = np.random.default_rng(npairs + n)
    # vertices outside [0, n) on both sides are ignored; whole-number
    # gradients make every sum exact in any order
    v = rng.integers(-2, n + 3, (2, npairs))
    v[:, : npairs // 3] = rng.integers(0, min(n, 50), (2, npairs // 3))
    g = rng.integers(-1000, 1000, (2, npairs)).astype(np.float64)
    want = np.zeros(n)
    inside = (v >= 0) & (v < n)
    np.add.at(want, v[inside], g[inside])
    codes = torch.from_numpy(v << 8 | rng.integers(0, 14, (2, npairs))).cuda()
    gt = torch.from_numpy(g).cuda()
    print("backward", npairs, n, flush=True)
    got = dms.gradient_backward(codes[0].contiguous(), codes[1].contiguous(), gt[0].contiguous(), gt[1].contiguous(), n)
    assert (got.cpu().numpy() == want).all()


@pytest.mark.parametrize("dims", [(5, 4, 3), (17, 13, 11), (64, 50, 41)])
@pytest.mark.parametrize("dim", [0, 1, 2, 3])
def test_sort_any_cells(dims, dim):
    nx, ny, nz = dims
    n = nx * ny * nz
    rng = np.random.default_rng(n + dim)
    order = rng.permutation(n).astype(np.int32)
    t = dms.star_tables()
    nb = t["nb"].astype(np.int64)
    star = [np.zeros((1, 0), np.int64), np.arange(14)[:, None], t["tri"].astype(np.int64), t["tet"].astype(np.int64)][dim]
    count = 4000 if n > 100 else 700
    v = rng.integers(0, n, count)
    loc = rng.integers(0, len(star), count)
    xyz = np.stack([v % nx, v // nx % ny, v // (nx * ny)], 1)
    oth = xyz[:, None, :] + nb[star[loc]]
    inside = ((oth >= 0) & (oth < np.array([nx, ny, nz]))).all(axis=(1, 2))
    v, loc, oth = v[inside], loc[inside], oth[inside]
    keys = np.concatenate([order[v][:, None], order[oth @ np.array([1, nx, nx * ny])]], 1).astype(np.int64)
    keys = -np.sort(-keys, axis=1)
    codes = v << 8 | loc
    want = codes[np.lexsort(keys.T[::-1])]  # stable: equal cells keep their order
    print("sort cells", dims, dim, codes.size, flush=True)
    got = dms.critical_sort(torch.from_numpy(codes).cuda(), dim, torch.from_numpy(order).cuda(), dims).cpu().numpy()
    assert (got == want).all()
    # codes naming no cell sort last, in their order, and are reported
    bad = np.array([n << 8, -1, (n + 7) << 8 | 1])
    mixed = np.concatenate([bad[:2], codes, bad[2:]])
    flags = dms.new_flags("cuda")
    got = dms.critical_sort(torch.from_numpy(mixed).cuda(), dim, torch.from_numpy(order).cuda(), dims, flags=flags,
                            check=False).cpu().numpy()
    assert int(flags.item()) == dms.FLAG_BADCODE
    assert (got == np.concatenate([want, bad])).all()
