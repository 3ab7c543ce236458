"""Timing cases of the neighbour search, through the package's public entry points.

A case is a plain dict; `prepare` makes what a program holds before the call (positions on
the GPU, a context, a cell structure, output buffers where a time loop would keep them),
`run` makes one pass and returns its outputs, `work` states the bytes and operations the
pass cannot do without, and `exact` gives the distances (and gradients) in plain binary64.

Kinds of case (the "kind" key):
  search   one search at a time on a reused cell structure: build, count (waits for the
           number of pairs), fill
  step     one graph-replayed build + count + fill of a time loop (Cells.batch_step)
  batch    the same over several sets of different sizes in one structure
  update   two incremental steps (displacements there and back) of a time loop
  allpairs one all-list search of a small set
  gradient one SPH gradient over a neighbour list

Programs that search again and again keep their lists in buffers with some room: columns
and distances are `_room` entries long here, zero past the last pair.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2401_08586_amd import nnps
from paper_2401_08586_amd import workloads as W

MODES = {"fp16": nnps.MODE_FP16_RCLL, "fp64": nnps.MODE_FP64_BASELINE, "fp32": nnps.MODE_FP32_RCLL}


def listed():
    return [
        # a few thousand particles: below the all-list crossover, where launches count
        {"name": "allpairs_3d_2k", "kind": "allpairs", "shape": "uniform", "dim": 3, "n": 2000},
        # the small 2D lattice of the benchmarks (100 x 100), one search at a time
        {"name": "search_2d_10k", "kind": "search", "shape": "lattice", "dim": 2, "n": 10000, "mode": "fp16"},
        # an odd-sized cloud with no order in its numbering, one search at a time
        {"name": "search_3d_64k", "kind": "search", "shape": "uniform", "dim": 3, "n": 64003, "mode": "fp16"},
        # the headline workload: 100^3 lattice, the step of a time loop
        {"name": "step_3d_1m", "kind": "step", "shape": "lattice", "dim": 3, "n": 1000000, "mode": "fp16", "half": False},
        # the same in binary64, the comparison of the headline
        {"name": "step_3d_1m_fp64", "kind": "step", "shape": "lattice", "dim": 3, "n": 1000000, "mode": "fp64",
         "half": False},
        # the large 2D lattice of the benchmarks (1000 x 1000)
        {"name": "step_2d_1m", "kind": "step", "shape": "lattice", "dim": 2, "n": 1000000, "mode": "fp16", "half": False},
        # single precision at a middle size (60^3)
        {"name": "step_3d_216k_fp32", "kind": "step", "shape": "lattice", "dim": 3, "n": 216000, "mode": "fp32",
         "half": False},
        # half lists (each pair once), for solvers that apply a pair to both sides; odd size (71^3)
        {"name": "step_3d_358k_half", "kind": "step", "shape": "lattice", "dim": 3, "n": 357911, "mode": "fp16",
         "half": True},
        # clustered sets of uneven size in one batch: long rows, dense cells
        {"name": "batch_clustered", "kind": "batch", "shape": "clustered", "dim": 3, "nsets": 6, "lo": 10000, "hi": 200000,
         "mode": "fp16"},
        # many small simulations stepped together, as a server batches them
        {"name": "batch_2d_small", "kind": "batch", "shape": "lattice", "dim": 2, "nsets": 16, "lo": 1000, "hi": 50000,
         "mode": "fp16"},
        # a simulation stepped by the incremental update
        {"name": "update_3d_250k", "kind": "update", "shape": "lattice", "dim": 3, "n": 250047, "mode": "fp16"},
        # the consumer of the list at the headline size
        {"name": "gradient_3d_1m", "kind": "gradient", "shape": "lattice", "dim": 3, "n": 1000000},
    ]


def _log(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def _mode(rng):
    return rng.choice(["fp16", "fp16", "fp16", "fp16", "fp64", "fp32"])


def draw(rng):
    kind = rng.choice(["search", "search", "step", "step", "step", "batch", "batch", "update", "allpairs", "gradient"])
    dim = rng.choice([2, 3])
    shape = rng.choice(["lattice", "uniform"])
    if kind == "allpairs":
        return {"kind": kind, "shape": shape, "dim": dim, "n": _log(rng, 500, 12000)}
    if kind == "search":
        return {"kind": kind, "shape": rng.choice(["lattice", "uniform", "clustered"]), "dim": dim,
                "n": _log(rng, 2000, 100000), "mode": _mode(rng)}
    if kind == "batch":
        if rng.random() < 0.5:
            return {"kind": kind, "shape": "clustered", "dim": dim, "nsets": rng.randint(1, 6),
                    "lo": _log(rng, 2000, 10000), "hi": _log(rng, 10000, 150000), "mode": "fp16"}
        return {"kind": kind, "shape": "lattice", "dim": dim, "nsets": rng.randint(4, 20),
                "lo": _log(rng, 1000, 5000), "hi": _log(rng, 5000, 50000), "mode": _mode(rng)}
    n = _log(rng, 10000, 1000000)
    if kind == "update":
        return {"kind": kind, "shape": shape, "dim": dim, "n": n, "mode": "fp16"}
    if kind == "gradient":
        return {"kind": kind, "shape": shape, "dim": dim, "n": n}
    return {"kind": kind, "shape": shape, "dim": dim, "n": n, "mode": _mode(rng), "half": rng.random() < 0.2}


def _sizes(case):
    """Particles per set: one set, or nsets sizes spaced evenly in the logarithm."""
    if "nsets" not in case:
        return [case["n"]]
    k = case["nsets"]
    return [int(round(case["lo"] * (case["hi"] / case["lo"]) ** (i / max(k - 1, 1)))) for i in range(k)]


def _sets(case, seed):
    dim, out = case["dim"], []
    for i, n in enumerate(_sizes(case)):
        s = 1000 * seed + i
        if case["shape"] == "lattice":
            side = max(2, int(round(n ** (1.0 / dim))))
            out.append(W.lattice(dim, side, 1.0 / side, 0.1, seed=s))
        elif case["shape"] == "uniform":
            out.append(W.uniform(dim, n, seed=s))
        else:
            out.append(_clustered(dim, n, s))
    return out


def _clustered(dim, n, seed):
    """W.clustered's mixture (a fifth uniform, the rest in eight Gaussian clusters) with the
    widths spread evenly over 0.02 .. 0.1 and the centres kept apart, so that every seed has
    about the same number of pairs."""
    rng = np.random.default_rng(seed)
    nbg = n // 5
    which = np.arange(n - nbg) % 8
    corner = np.stack([(np.arange(8) >> k) & 1 for k in range(dim)], axis=1) if dim == 3 else \
        np.stack([np.cos(np.arange(8) * math.pi / 4), np.sin(np.arange(8) * math.pi / 4)], axis=1) * 0.5 + 0.5
    centres = 0.25 + 0.5 * corner + rng.uniform(-0.05, 0.05, size=(8, dim))
    sig = rng.permutation(0.025 + 0.01 * np.arange(8))
    pts = centres[which] + rng.standard_normal((n - nbg, dim)) * sig[which, None]
    while True:
        out = np.any((pts < 0.0) | (pts > 1.0), axis=1)
        if not out.any():
            break
        pts[out] = centres[which[out]] + rng.standard_normal((int(out.sum()), dim)) * sig[which[out], None]
    pos = np.concatenate([rng.uniform(0.0, 1.0, size=(nbg, dim)), pts])[rng.permutation(n)]
    r = 2.4 * (1.0 / n) ** (1.0 / dim)
    return W.ParticleSet(np.ascontiguousarray(pos), (0.0,) * dim, (1.0,) * dim, r, r)


def _particles(case):
    if case["shape"] != "lattice":
        return _sizes(case)
    return [max(2, int(round(n ** (1.0 / case["dim"])))) ** case["dim"] for n in _sizes(case)]


def _per_set(case):
    """Expected neighbour pairs of each set: a radius ball of 2.4 spacings (a perfect
    lattice's shells in the interior); clustered sets about 1600 (3D) or 75 (2D) a particle."""
    ball = {("lattice", 2): 20, ("lattice", 3): 56, ("uniform", 2): 18, ("uniform", 3): 58, ("clustered", 2): 75,
            ("clustered", 3): 1600}[case["shape"], case["dim"]]
    return [n * ball * (0.5 if case.get("half") else 1.0) for n in _particles(case)]


def _pairs(case):
    return sum(_per_set(case))


def _room(case):
    return [int(1.25 * k) + 64 for k in _per_set(case)]


def _fixed(ps, amp):
    """Positions and displacements on a grid of 2^-40, so that moving there and back is exact."""
    q = 2.0 ** 40
    pos = np.round(ps.pos * q) / q
    return pos, lambda seed: np.round(W.reflected_displacement(pos, ps.lo, ps.hi, amp, seed) * q) / q


def _field(pos):
    return torch.sin(7.0 * pos[:, 0]) + pos[:, 1] * pos[:, 1] + 0.25 * torch.cos(5.0 * pos[:, -1])


def _moves(case, seed):
    ps = _sets(case, seed)[0]
    pos, disp = _fixed(ps, 0.05 * ps.radius / 2.4)
    return ps, pos, disp(seed + 77)


def prepare(case, seed):
    kind = case["kind"]
    mode = MODES[case.get("mode", "fp16")]
    ctx = nnps.Context(0)
    if kind == "update":
        ps, pos, d = _moves(case, seed)
        pss = [ps]
        pos = [torch.from_numpy(pos).cuda()]
    else:
        pss = _sets(case, seed)
        pos = [torch.from_numpy(p.pos).cuda() for p in pss]
    sets = [(x, p.lo, p.hi, p.cell_size, p.radius) for x, p in zip(pos, pss)]
    st = {"case": case, "ctx": ctx, "sets": sets, "mode": mode}
    rps = [torch.empty(x.shape[0] + 1, dtype=torch.int64, device="cuda") for x in pos]
    cols = [torch.zeros(k, dtype=torch.int32, device="cuda") for k in _room(case)]
    dists = [torch.zeros(k, dtype=torch.float32, device="cuda") for k in _room(case)]
    st.update(rps=rps, cols=cols, dists=dists)
    if kind == "allpairs":
        return st
    # the structure a program has from its searches before: its buffers are grown, and the
    # lists are known to fit
    cells = st["cells"] = ctx.cells()
    cells.set_half(bool(case.get("half")))
    cells.batch_build(sets, mode)
    nnz = cells.batch_count(rps)
    assert all(k <= c.numel() for k, c in zip(nnz, cols)), "the lists' room is too small"
    cells.batch_fill(rps, cols, dists)
    if kind == "gradient":
        st.update(f=_field(pos[0]), h=pss[0].radius / 2.0, col=cols[0][:nnz[0]].clone())
        torch.cuda.synchronize()
        cells.close()
        return st
    if kind == "search":
        return st
    st["stream"] = torch.cuda.Stream()
    cells.set_graphs(True)
    if kind == "update":
        cols[0].zero_()  # the moved positions' list may be the shorter one
        dists[0].zero_()
        st.update(disp=[torch.from_numpy(d).cuda(), torch.from_numpy(-d).cuda()],
                  rps2=[torch.empty_like(t) for t in rps], cols2=[torch.zeros_like(t) for t in cols],
                  dists2=[torch.zeros_like(t) for t in dists])
    torch.cuda.synchronize()
    return st


def run(st):
    kind = st["case"]["kind"]
    if kind == "allpairs":
        pos, lo, hi, _, radius = st["sets"][0]
        nnps.allpairs_search_noalloc(pos, lo, hi, radius, st["rps"][0], st["cols"][0], st["dists"][0], st["ctx"])
        return [st["rps"][0], st["cols"][0], st["dists"][0]]
    if kind == "gradient":
        x = st["sets"][0][0]
        return list(nnps.sph_gradient(x, st["f"], st["h"], st["rps"][0], st["col"], ctx=st["ctx"]))
    if kind == "search":
        cells = st["cells"]
        cells.build(*st["sets"][0], mode=st["mode"])
        cells.count(st["rps"][0])
        cells.fill(st["rps"][0], st["cols"][0], st["dists"][0])
        return [st["rps"][0], st["cols"][0], st["dists"][0]]
    cells, stream = st["cells"], st["stream"]
    if kind == "update":
        cells.batch_update_step(st["rps"], st["cols"], st["dists"], disp=st["disp"][0], stream=stream)
        cells.batch_update_step(st["rps2"], st["cols2"], st["dists2"], disp=st["disp"][1], stream=stream)
        return [st["sets"][0][0], st["rps"], st["cols"], st["dists"], st["rps2"], st["cols2"], st["dists2"]]
    cells.batch_step(st["sets"], st["rps"], st["cols"], st["dists"], st["mode"], stream=stream)
    return [st["rps"], st["cols"], st["dists"]]


def work(case):
    """Positions read once and the CSR (8 bytes a pair, 8 a row) written once; a distance test
    per pair that comes out (3 dim operations). The gradient reads the list, positions and
    field and writes two vectors; the update also reads displacements and writes positions."""
    n, pairs, d = sum(_particles(case)), _pairs(case), case["dim"]
    if case["kind"] == "gradient":
        return {"bytes": n * (8 * d + 8 + 8 + 16 * d) + 4 * pairs, "flops": pairs * (12 * d + 12)}
    if case["kind"] == "allpairs":
        return {"bytes": n * (8 * d + 8) + 8 * pairs, "flops": float(n) * n * 3 * d}
    one = {"bytes": n * (8 * d + 8) + 8 * pairs, "flops": pairs * 3 * d}
    if case["kind"] == "update":
        return {"bytes": 2 * (one["bytes"] + 16 * d * n), "flops": 2 * one["flops"]}
    return one


def _plain_lists(pos, lo, radius, half):
    """Rows, columns and squared distances of every pair within the radius, rows and columns
    ascending: particles sorted into square cells, the rows of cells around each tested."""
    n, dim = pos.shape
    dev = pos.device
    c = torch.floor((pos - torch.tensor(lo, dtype=torch.float64, device=dev)) / (radius * (1 + 1e-9))).to(torch.int64)
    nc = [int(c[:, k].max()) + 1 for k in range(dim)]
    ny, nz = nc[1], nc[2] if dim == 3 else 1
    key = c[:, 0] + nc[0] * (c[:, 1] + (ny * c[:, 2] if dim == 3 else 0))
    order = torch.argsort(key)
    start = torch.zeros(nc[0] * ny * nz + 1, dtype=torch.int64, device=dev)
    start[1:] = torch.cumsum(torch.bincount(key, minlength=nc[0] * ny * nz), 0)
    sp = pos[order]
    keys, r2s = [], []
    xa, xb = torch.clamp(c[:, 0] - 1, min=0), torch.clamp(c[:, 0] + 1, max=nc[0] - 1)
    for dz in ((-1, 0, 1) if dim == 3 else (0,)):
        for dy in (-1, 0, 1):
            yy = c[:, 1] + dy
            zz = (c[:, 2] if dim == 3 else torch.zeros_like(yy)) + dz
            ok = (yy >= 0) & (yy < ny) & (zz >= 0) & (zz < nz)
            base = nc[0] * (yy + ny * zz) * ok
            a = torch.where(ok, start[base + xa * ok], torch.zeros_like(base))
            m = torch.where(ok, start[(base + xb) * ok + 1], a) - a
            ends = torch.cumsum(m, 0)
            i0, done = 0, 0
            while i0 < n:  # about 2^27 candidates at a time
                i1 = max(i0 + 1, int(torch.searchsorted(ends, torch.tensor(done + (1 << 27), device=dev), right=True)))
                mm = m[i0:i1]
                tot = int(mm.sum())
                rows = torch.repeat_interleave(torch.arange(i0, i1, device=dev), mm, output_size=tot)
                off = torch.arange(tot, device=dev) - torch.repeat_interleave(torch.cumsum(mm, 0) - mm, mm, output_size=tot)
                j = a[rows] + off
                e = sp[j] - pos[rows]
                e = e * e
                r2 = e[:, 0] + e[:, 1]
                if dim == 3:
                    r2 = r2 + e[:, 2]
                cols = order[j]
                keep = (r2 <= radius * radius) & ((cols > rows) if half else (cols != rows))
                keys.append(rows[keep] * n + cols[keep])
                r2s.append(r2[keep])
                done, i0 = int(ends[i1 - 1]), i1
    keys = torch.cat(keys)
    at = torch.argsort(keys)
    keys = keys[at]
    return keys // n, keys % n, torch.cat(r2s)[at]


def _plain_gradient(pos, f, h, rows, cols, r2):
    n, dim = pos.shape
    alpha = 15.0 / (7.0 * math.pi * h * h) if dim == 2 else 3.0 / (2.0 * math.pi * h ** 3)
    r = torch.sqrt(r2)
    q = r / h
    dw = torch.where(q < 1, -2 * q + 1.5 * q * q, torch.where(q < 2, -0.5 * (2 - q) ** 2, torch.zeros_like(q)))
    g = torch.where(r > 0, alpha / h * dw / r, torch.zeros_like(r))
    add = lambda v: torch.zeros(n, dtype=torch.float64, device=pos.device).index_add_(0, rows, v)  # noqa: E731
    grad, norm = [], []
    for k in range(dim):
        dx = pos[cols, k] - pos[rows, k]
        grad.append(add(-f[cols] * g * dx))
        den = add(-dx * dx * g)
        norm.append(torch.where(den != 0, add(-(f[cols] - f[rows]) * g * dx) / den, torch.zeros_like(den)))
    return [torch.stack(grad, 1), torch.stack(norm, 1)]


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    half = bool(case.get("half"))

    def dist(pos, ps, size):
        r = torch.sqrt(_plain_lists(pos, ps.lo, ps.radius, half)[2])
        return torch.cat([r, torch.zeros(size - r.numel(), dtype=r.dtype, device=dev)])

    room = _room(case)
    if case["kind"] == "update":
        ps, pos, d = _moves(case, seed)
        pos, d = torch.from_numpy(pos).to(dev), torch.from_numpy(d).to(dev)
        return [pos, [None], [None], [dist(pos + d, ps, room[0])], [None], [None], [dist(pos, ps, room[0])]]
    pss = _sets(case, seed)
    pos = [torch.from_numpy(p.pos).to(dev) for p in pss]
    if case["kind"] == "gradient":
        rows, cols, r2 = _plain_lists(pos[0], pss[0].lo, pss[0].radius, False)
        return _plain_gradient(pos[0], _field(pos[0]), pss[0].radius / 2.0, rows, cols, r2)
    if "nsets" in case or case["kind"] == "step":
        return [[None] * len(pss), [None] * len(pss), [dist(x, p, k) for x, p, k in zip(pos, pss, room)]]
    return [None, None, dist(pos[0], pss[0], room[0])]
