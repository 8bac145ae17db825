"""The workloads whose speed is followed: what users of the library have it do.

listed() gives the fixed cases and draw() further ones of the same ranges;
prepare() makes what a program holds before the call (the field on the GPU,
kept buffers, a batch handle), run() is one pass through the public entry
points, work() the bytes a pass cannot do without, and exact() the outputs
that plain torch gives in 64 bits (None where there is no such value).

A case's "kind" is the call a program makes:
  pipe     gradient_pipeline: order, records and exact critical lists of a
           field that comes once (lists sized by the counting call)
  step     the same three stages on kept buffers, for a time loop: order,
           gradient of the owned box with the critical mask, masked extraction
  values   the gradient straight from the values (no order), then the
           extraction with the library's own scratch: the serving form
  batch    Batch.run over many uneven fields (an ensemble)
  persist  PersistenceD0 / PersistenceD2: pairs of a field, a loss on their
           persistence and its gradient with respect to the field
  sort     critical_sort of the four critical lists and the cells' values
Fields are white noise (the "noise" field: every vertex irregular) or a
mixture of Gaussian bumps plus small noise ("mix": mostly regular vertices).
A program keeps one table of critical cells (or pairs) with room for "room"
of them per vertex, and stores a pass's lists in it one after the other.
"""
import math

import numpy as np
import torch

import paper_2505_21266_amd as dms
from paper_2505_21266_amd.autograd import d0_loss

_TORCH = {"f32": torch.float32, "f64": torch.float64}
_EXACT_ORDER = 1 << 25   # largest field whose order is checked against a 64-bit sort
_EXACT_PAIRS = 60000     # largest field whose pairs are checked against a sweep over its vertices


def listed():
    return [
        # a first call on a small block: latency and launches
        dict(name="pipe_tiny", kind="pipe", nx=24, ny=20, nz=16, dtype="f32", field="noise", bumps=0, noise=1.0,
             room=0.8),
        # the 64^3 white-noise block
        dict(name="pipe_noise64", kind="pipe", nx=64, ny=64, nz=64, dtype="f32", field="noise", bumps=0, noise=1.0,
             room=0.8),
        # an ordinary double-precision simulation block with odd sides
        dict(name="pipe_f64_odd", kind="pipe", nx=131, ny=97, nz=75, dtype="f64", field="mix", bumps=16, noise=1e-4,
             room=0.4),
        # one time step of a noisy 512^3 simulation, buffers kept
        dict(name="step_mix512", kind="step", nx=512, ny=512, nz=512, ghost=0, dtype="f32", field="mix", bumps=64,
             noise=1e-3, room=0.4),
        # one GPU's share of a distributed run: 1024^3 owned with a ghost layer
        dict(name="step_ghost1026", kind="step", nx=1026, ny=1026, nz=1026, ghost=1, dtype="f32", field="mix",
             bumps=512, noise=1e-3, room=0.004),
        # a smooth scan served without its order, single precision, ragged sides
        dict(name="values_f32", kind="values", nx=643, ny=511, nz=386, ghost=1, dtype="f32", field="mix", bumps=64,
             noise=1e-3, room=0.4),
        # the same in double precision
        dict(name="values_f64", kind="values", nx=259, ny=257, nz=194, ghost=0, dtype="f64", field="mix", bumps=32,
             noise=1e-4, room=0.2),
        # an ensemble of 96 fields with sides 32..256, half noise, half mixtures
        dict(name="batch96", kind="batch", nfields=96, lo=32, hi=256, room=0.5),
        # a few small ensemble members
        dict(name="batch_small", kind="batch", nfields=12, lo=7, hi=40, room=0.6),
        # topological loss on components of a 128^3 double-precision field, forward and backward
        dict(name="persist_d0", kind="persist", dim=0, nx=128, ny=128, nz=128, dtype="f64", field="mix", bumps=16,
             noise=1e-4, room=0.125),
        # the same on voids, of a single-precision field with uneven sides
        dict(name="persist_d2", kind="persist", dim=2, nx=112, ny=80, nz=96, dtype="f32", field="mix", bumps=16,
             noise=1e-3, room=0.125),
        # filtration-ordered critical cells of a 256^3 field
        dict(name="sort_mix256", kind="sort", nx=256, ny=256, nz=256, dtype="f32", field="mix", bumps=64,
             noise=1e-3, room=0.4),
    ]


def _sides(rng, lo, hi):
    """Three uneven sides whose product lies about log-uniformly in [lo, hi]."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    r = [math.exp(rng.uniform(-0.5, 0.5)) for _ in range(3)]
    s = (n / (r[0] * r[1] * r[2])) ** (1.0 / 3.0)
    return {k: max(2, int(round(s * f))) for k, f in zip(("nx", "ny", "nz"), r)}


def _field_kind(rng, dtype):
    if rng.random() < 0.35:
        return dict(field="noise", bumps=0, noise=1.0)
    return dict(field="mix", bumps=rng.choice([8, 16, 32, 64]),
                noise=rng.choice([1e-3, 1e-4]) if dtype == "f32" else 1e-4)


def draw(rng):
    kind = rng.choice(["pipe", "pipe", "step", "values", "batch", "persist", "sort"])
    dtype = "f32" if rng.random() < 0.65 else "f64"
    c = dict(kind=kind)
    if kind == "batch":
        c["nfields"] = rng.randint(2, 80)
        c["lo"] = rng.randint(4, 40)
        c["hi"] = c["lo"] + rng.randint(8, 160)
        c["room"] = 0.6
        return c
    top = {"pipe": 1 << 26, "step": 1 << 28, "values": 1 << 27, "persist": 1 << 21, "sort": 1 << 24}[kind]
    if dtype == "f64":
        top >>= 1
    c.update(_sides(rng, 4000, top))
    c.update(dtype=dtype, **_field_kind(rng, dtype))
    if kind in ("step", "values"):
        c["ghost"] = rng.randint(0, 1)
    if kind == "persist":
        c["dim"] = rng.choice([0, 2])
    c["room"] = 0.125 if kind == "persist" else 0.8 if c["field"] == "noise" else 0.5
    return c


# ------------------------------------------------------------------ inputs


def _field(shape, dtype, field, bumps, noise, gen, dev):
    """A (nz, ny, nx) field on the GPU from the generator alone: U[0, 1) noise,
    or `bumps` isotropic Gaussians (sigma 0.02..0.1, amplitude -1..1) plus
    noise * U[0, 1)."""
    t = _TORCH[dtype]
    out = torch.rand(shape, generator=gen, device=dev, dtype=t)
    if field == "noise":
        return out
    out.mul_(noise)
    par = torch.rand((bumps, 5), generator=gen, device=dev, dtype=torch.float64)
    sigma = 0.02 + 0.08 * par[:, 3]
    amp = 2.0 * par[:, 4] - 1.0
    axes = []
    for n, col in zip(shape, (2, 1, 0)):
        x = torch.arange(n, device=dev, dtype=torch.float64) / max(n - 1, 1)
        axes.append(torch.exp(-(x[None, :] - par[:, col, None]) ** 2 / (2.0 * sigma[:, None] ** 2)))
    fz, fy, fx = (axes[0] * amp[:, None]).to(t), axes[1].to(t), axes[2].to(t)
    for b in range(bumps):
        out.addcmul_((fz[b][:, None] * fy[b][None, :])[:, :, None], fx[b][None, None, :])
    return out


def _shape(case):
    return (case["nz"], case["ny"], case["nx"])


def _batch_sides(case):
    return np.random.default_rng(4).integers(case["lo"], case["hi"] + 1, (case["nfields"], 3))


def _vertices(case):
    if case["kind"] == "batch":
        return int(_batch_sides(case).prod(axis=1).sum())
    return case["nx"] * case["ny"] * case["nz"]


def _room(case):
    return int(case["room"] * _vertices(case)) + 64


def _store(table, lists):
    """The lists one after the other at the front of the kept table."""
    used = sum(t.numel() for t in lists)
    if used > table.numel():
        raise RuntimeError("the kept table is too small: %d cells" % used)
    torch.cat(lists, out=table[:used])
    return table


def _inputs(case, seed):
    """The values a case works on: a field, or a batch's fields concatenated."""
    dev = torch.device("cuda", torch.cuda.current_device())
    gen = torch.Generator(device=dev)
    gen.manual_seed(1000003 * (seed + 1))
    if case["kind"] != "batch":
        return _field(_shape(case), case["dtype"], case["field"], case["bumps"], case["noise"], gen, dev)
    parts = []
    for f, (nx, ny, nz) in enumerate(_batch_sides(case).tolist()):
        kind = ("noise", 0, 1.0) if f % 2 == 0 else ("mix", 16, 1e-3)
        parts.append(_field((nz, ny, nx), "f32", *kind, gen, dev).reshape(-1))
    return torch.cat(parts)


def _box(case):
    g = case["ghost"] if min(case["nx"], case["ny"], case["nz"]) > 2 else 0
    return (g, g, g), (case["nx"] - g, case["ny"] - g, case["nz"] - g)


def prepare(case, seed):
    values = _inputs(case, seed)
    dev = values.device
    s = dict(case=case, values=values)
    kind = case["kind"]
    if kind == "batch":
        s["batch"] = dms.Batch([tuple(int(x) for x in d) for d in _batch_sides(case)])
    elif kind in ("step", "values"):
        # the buffers that a time loop or a server keeps
        lo, hi = _box(case)
        dims = dms.dims_of(values)
        nbox = (hi[0] - lo[0]) * (hi[1] - lo[1]) * (hi[2] - lo[2])
        s.update(lo=lo, hi=hi, dims=dims, rec=torch.empty((nbox, 4), dtype=torch.int32, device=dev),
                 mask=dms.critical_mask(nbox, dev), gws=dms.gradient_workspace(values, lo, hi),
                 flags=dms.new_flags(dev), counts=torch.zeros(4, dtype=torch.int64, device=dev))
        if kind == "step":
            # the lists are as long as one earlier pass over this field found
            s["order"] = torch.empty(values.shape, dtype=torch.int32, device=dev)
            dms.discrete_gradient_values(values, lo, hi, out=s["rec"], workspace=s["gws"], mask=s["mask"])
            _, counts = dms.critical_simplices(s["rec"], dims, lo, hi, mask=s["mask"])
            s["cap"] = counts.cpu().numpy().copy()
        else:
            s["cap"] = np.full(4, _room(case), np.int64)
            s["lists"] = [torch.zeros(_room(case), dtype=torch.int64, device=dev) for _ in range(4)]
    elif kind == "sort":
        s["dims"] = dms.dims_of(values)
        s["order"], _, s["lists"], _ = dms.gradient_pipeline(values)
        s["values_out"] = torch.zeros(_room(case), dtype=torch.float64, device=dev)
    if kind == "persist":
        s["table"] = torch.zeros((2, _room(case)), dtype=values.dtype, device=dev)
    elif kind != "values":
        s["table"] = torch.zeros(_room(case), dtype=torch.int64, device=dev)
    return s


def run(s):
    case, values = s["case"], s["values"]
    kind = case["kind"]
    if kind == "pipe":
        order, rec, lists, counts = dms.gradient_pipeline(values)
        return order, rec, _store(s["table"], lists), counts
    if kind == "step":
        dms.order(values, out=s["order"], flags=s["flags"], check=False)
        dms.discrete_gradient(s["order"], s["lo"], s["hi"], out=s["rec"], workspace=s["gws"], mask=s["mask"])
        lists, counts = dms.critical_simplices(s["rec"], s["dims"], s["lo"], s["hi"], cap=s["cap"], flags=s["flags"],
                                               counts=s["counts"], mask=s["mask"])
        return s["order"], s["rec"], _store(s["table"], lists), counts, s["flags"]
    if kind == "values":
        dms.discrete_gradient_values(values, s["lo"], s["hi"], out=s["rec"], workspace=s["gws"], flags=s["flags"],
                                     check=False, mask=s["mask"])
        lists, counts = dms.critical_simplices_noalloc(s["rec"], s["dims"], s["cap"], s["lo"], s["hi"],
                                                       lists=s["lists"], counts=s["counts"], flags=s["flags"],
                                                       mask=s["mask"])
        return s["rec"], lists, counts, s["flags"]
    if kind == "batch":
        order, rec, lists, counts, offsets = s["batch"].run(values)
        return order, rec, _store(s["table"], lists), counts, offsets
    if kind == "persist":
        x = values.detach().requires_grad_()
        births, deaths = (dms.PersistenceD0 if case["dim"] == 0 else dms.PersistenceD2).apply(x)
        d0_loss(births, deaths).backward()
        torch.stack((births.detach(), deaths.detach()), out=s["table"][:, :births.numel()])
        return s["table"], x.grad
    at = 0
    for d in range(4):
        k = s["lists"][d].numel()
        cells = dms.critical_sort(s["lists"][d], d, s["order"], s["dims"], out=s["table"][at:at + k])
        dms.simplex_values(values, cells, out=s["values_out"][at:at + k])
        at += k
    return s["table"], s["values_out"]


def work(case):
    """Bytes of inputs read once and outputs written once (4-byte orders,
    16-byte records; the critical cells' share is small or unknown beforehand).
    There is no floating-point arithmetic to count."""
    n = _vertices(case)
    if case["kind"] == "batch":
        return {"bytes": n * (4 + 4 + 16), "flops": 0}
    v = 4 if case["dtype"] == "f32" else 8
    if case["kind"] in ("pipe", "step"):
        return {"bytes": n * (v + 4 + 16), "flops": 0}
    if case["kind"] == "values":
        return {"bytes": n * (v + 16), "flops": 0}
    if case["kind"] == "persist":
        return {"bytes": n * 2 * v, "flops": 0}
    return {"bytes": n // 64 * 24, "flops": 0}


# ------------------------------------------------------- 64-bit outputs


def _order64(values):
    flat = values.reshape(-1).double()
    perm = torch.sort(flat, stable=True).indices
    out = torch.empty_like(perm)
    out[perm] = torch.arange(perm.numel(), device=perm.device)
    return out.reshape(values.shape)


def _pairs64(values):
    """D0 pairs by a sweep over the vertices in order: a vertex joins the
    component of its lowest neighbour, and every further component among its
    lower neighbours (in order) is merged, the later-born minimum dying here."""
    f = values.reshape(-1).double().cpu().numpy()
    order = _order64(values).reshape(-1).cpu().numpy()
    nz, ny, nx = values.shape
    steps = [tuple(int(c) for c in d) for d in dms.star_tables()["nb"]]
    parent, birth = list(range(f.size)), list(range(f.size))

    def root(a):
        while parent[a] != a:
            parent[a] = parent[parent[a]]
            a = parent[a]
        return a

    pairs = []
    for v in np.argsort(order).tolist():
        x, y, z = v % nx, v // nx % ny, v // (nx * ny)
        low = []
        for dx, dy, dz in steps:
            if 0 <= x + dx < nx and 0 <= y + dy < ny and 0 <= z + dz < nz:
                u = x + dx + nx * (y + dy + ny * (z + dz))
                if order[u] < order[v]:
                    low.append((order[u], u))
        for k, (_, u) in enumerate(sorted(low)):
            a, b = root(v), root(u)
            if k == 0:
                parent[a] = b
            elif a != b:
                if order[birth[a]] < order[birth[b]]:
                    a, b = b, a
                pairs.append((birth[a], v))
                parent[a] = b
    return f, np.asarray(pairs, dtype=np.int64).reshape(-1, 2)


def exact(case, seed):
    kind, n = case["kind"], _vertices(case)
    if kind in ("batch", "pipe", "step") and n <= _EXACT_ORDER:
        values = _inputs(case, seed)
        if kind == "batch":
            sizes = _batch_sides(case).prod(axis=1).tolist()
            return torch.cat([_order64(p) for p in torch.split(values, sizes)]), None, None, None, None
        return (_order64(values), None, None, None) + ((None,) if kind == "step" else ())
    if kind == "persist" and case["dim"] == 0 and n <= _EXACT_PAIRS:
        values = _inputs(case, seed)
        f, pairs = _pairs64(values)
        table = np.zeros((2, _room(case)))
        table[0, :len(pairs)], table[1, :len(pairs)] = f[pairs[:, 0]], f[pairs[:, 1]]
        pers = f[pairs[:, 1]] - f[pairs[:, 0]]
        g = 2.0 * pers * (pers < 0.05)
        grad = np.zeros(f.size)
        np.add.at(grad, pairs[:, 1], g)
        np.subtract.at(grad, pairs[:, 0], g)
        return torch.from_numpy(table), torch.from_numpy(grad).reshape(values.shape)
    return None
