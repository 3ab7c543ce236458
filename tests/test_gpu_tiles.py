"""The matrix-core count and the ranked fill at the sizes where they can go wrong: unions of
31 to 65 candidates and up to the union limit (1024 in 3D, 512 in 2D) and past it, blocks of
1 to 64 targets, rows of one candidate to nearly the whole union, sparse sets whose blocks span
many cells, numberings of every spread (one bitmap, two-level bitmap, sorted keys), pairs far
closer than a cell, boxes far from 0 and very small or large cells. Rows against the CPU
oracle: neighbours bit-identical, distances bit-identical in the binary64 modes and within
1e-6 relative (the documented bound) in the others, full and half lists."""
import numpy as np
import pytest

import oracle
from paper_2401_08586_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2401_08586_amd import nnps  # noqa: E402

MODES = {"fp16": nnps.MODE_FP16_RCLL, "fp64": nnps.MODE_FP64_BASELINE, "fp32": nnps.MODE_FP32_RCLL,
         "recheck_all": nnps.MODE_RECHECK_ALL}


def blob(n, dim, seed, cell=1.0, lo=0.0, scale=1.0, ncell=5, spread=None):
    """n points in the middle cell of an ncell^dim grid (every point in one union), radius the cell."""
    rng = np.random.default_rng(seed)
    pos = (ncell // 2 + rng.uniform(0.02, 0.98, size=(n, dim))) * cell
    pos = lo + scale * pos
    hi = lo + scale * ncell * cell
    return W.ParticleSet(pos, (lo,) * dim, (hi,) * dim, scale * cell, 0.7 * scale * cell, f"blob{dim}d_{n}_{lo}_{scale}")


def far_numbers(ps, stride, total, seed):
    """ps among `total` points, its particles numbered `stride` apart: the rest fill a distant part of the box."""
    rng = np.random.default_rng(seed)
    dim = ps.dim
    hi = np.asarray(ps.hi) + 40 * ps.cell_size
    pos = np.asarray(ps.hi) + rng.uniform(2.0, 39.0, size=(total, dim)) * ps.cell_size
    at = np.arange(ps.n) * stride
    pos[at] = ps.pos
    return W.ParticleSet(np.ascontiguousarray(pos), ps.lo, tuple(hi), ps.cell_size, ps.radius, f"{ps.name}_x{stride}")


def cases():
    out = []
    for dim in (2, 3):
        for n in (1, 2, 31, 32, 33, 63, 64, 65, 127, 129, 257, 511, 512, 513) + ((1023, 1024, 1025) if dim == 3 else ()):
            out.append(blob(n, dim, n))
        out.append(blob(200, dim, 5, lo=1.0e6, scale=1e-3))    # far from 0: few bits left in a cell
        out.append(blob(200, dim, 6, scale=1e-30))             # quantum outside FP32's range
        out.append(blob(200, dim, 7, scale=1e30))
        rng = np.random.default_rng(dim)
        # sparse: fewer than one particle in ten cells, so that blocks span many cells
        pos = rng.uniform(0, 1, size=(3000, dim))
        r = 0.2 * (1.0 / 3000) ** (1.0 / dim)
        out.append(W.ParticleSet(pos, (0.0,) * dim, (1.0,) * dim, r, r, f"sparse{dim}d"))
        # pairs at 1e-12 to 0.3 of the radius
        a = rng.uniform(0.1, 0.9, size=(1500, dim))
        d = rng.standard_normal((1500, dim))
        d *= (0.05 * 10.0 ** rng.uniform(-12, -0.5, size=1500) / np.linalg.norm(d, axis=1))[:, None]
        out.append(W.ParticleSet(np.concatenate([a, a + d]), (0.0,) * dim, (1.0,) * dim, 0.05, 0.05, f"near{dim}d"))
    b = blob(300, 3, 8)
    out += [far_numbers(b, 100, 40000, 1), far_numbers(b, 400, 130000, 2), far_numbers(b, 1000, 300000, 3)]
    return out


def half_of(rp, col, dist):
    rows = np.repeat(np.arange(len(rp) - 1), np.diff(rp))
    keep = col > rows
    h = np.zeros(len(rp), dtype=np.int64)
    np.cumsum(np.bincount(rows[keep], minlength=len(rp) - 1), out=h[1:])
    return h, col[keep], dist[keep]


@pytest.mark.parametrize("half", [False, True], ids=["full", "half"])
@pytest.mark.parametrize("mode", MODES)
def test_tiles_against_the_oracle(mode, half):
    ctx = nnps.Context(0)
    try:
        ctx.set_tuning(dense_min_union=-1)  # the block and long-row paths only
        for ps in cases():
            print(f"[gpu] tiles {ps.name} n={ps.n} {mode} half={half}", flush=True)
            want = oracle.search_ps(ps)
            if half:
                want = half_of(*want)
            cells = ctx.cells()
            cells.set_half(half)
            rp, col, dist, _ = nnps.search(torch.from_numpy(np.ascontiguousarray(ps.pos)).cuda(), ps.lo, ps.hi,
                                           ps.cell_size, ps.radius, mode=MODES[mode], ctx=ctx, cells=cells)
            cells.stats()
            np.testing.assert_array_equal(rp.cpu().numpy(), want[0], err_msg=ps.name)
            np.testing.assert_array_equal(col.cpu().numpy(), want[1], err_msg=ps.name)
            d = dist.cpu().numpy()
            if mode in ("fp64", "fp32"):
                np.testing.assert_array_equal(d.view(np.uint32), want[2].view(np.uint32), err_msg=ps.name)
            else:
                w = want[2].astype(np.float64)
                assert np.all(np.abs(d - w) <= 1e-6 * w), ps.name
            cells.close()
    finally:
        ctx.set_tuning()
        ctx.close()


@pytest.mark.parametrize("half", [False, True], ids=["full", "half"])
@pytest.mark.parametrize("mode", MODES)
def test_dense_tiles_against_the_oracle(mode, half):
    """Every cell through the dense-cell path: lists at the edges of a step (64 candidates), a
    kept-bits row (1024) and a staged chunk (2048, 4096), units at the edges of a wavefront
    and a slice (256 targets). The first search tests in the fill, the later ones take the
    count's bits; both give the oracle's rows, and the same distances bit for bit."""
    ctx = nnps.Context(0)
    try:
        ctx.set_tuning(dense_min_union=1)
        pss = [blob(n, dim, 100 + n) for dim in (2, 3) for n in (2, 63, 64, 65, 255, 256, 257, 1024, 1025, 2049, 4097)]
        pss += [p for p in cases() if p.name.startswith("near") or "_1e-30" in p.name or "_1000000" in p.name]
        for ps in pss:
            print(f"[gpu] dense tiles {ps.name} n={ps.n} {mode} half={half}", flush=True)
            want = oracle.search_ps(ps)
            if half:
                want = half_of(*want)
            pos = torch.from_numpy(np.ascontiguousarray(ps.pos)).cuda()
            cells = ctx.cells()
            cells.set_half(half)
            first = None
            for rep in range(2):
                rp, col, dist, _ = nnps.search(pos, ps.lo, ps.hi, ps.cell_size, ps.radius, mode=MODES[mode], ctx=ctx,
                                               cells=cells)
                assert cells.stats()["dense_rows"] > 0
                np.testing.assert_array_equal(rp.cpu().numpy(), want[0], err_msg=ps.name)
                np.testing.assert_array_equal(col.cpu().numpy(), want[1], err_msg=ps.name)
                d = dist.cpu().numpy()
                if mode in ("fp64", "fp32"):
                    np.testing.assert_array_equal(d.view(np.uint32), want[2].view(np.uint32), err_msg=ps.name)
                else:
                    w = want[2].astype(np.float64)
                    assert np.all(np.abs(d - w) <= 1e-6 * w), ps.name
                if rep:
                    np.testing.assert_array_equal(d, first, err_msg=ps.name)
                first = d
            cells.close()
    finally:
        ctx.set_tuning()
        ctx.close()
