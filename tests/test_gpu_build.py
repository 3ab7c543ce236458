"""The build's tables and the row pointers at the sizes where they can go wrong: scan tiles
(4096 elements; 16 and 1024 of them, where the way a tile finds its offset changes), sets
that begin, end or are empty inside a tile, outputs on any 8-byte address, grids with more
row segments than the block table's workgroups add up themselves (8192), blocks cut by a
full wavefront, the span and dense cells; and counts and fills that follow one another
without a build in between. Rows against the CPU oracle or a lattice's known rows, equal."""
import numpy as np
import pytest

import oracle
from paper_2401_08586_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2401_08586_amd import nnps  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    c = nnps.Context(0)
    yield c
    c.set_tuning()
    c.close()


def uniform(n, dim, seed, r=None):
    rng = np.random.default_rng(seed)
    r = 0.9 * (1.0 / max(n, 8)) ** (1.0 / dim) if r is None else r
    return W.ParticleSet(rng.uniform(0, 1, size=(n, dim)), (0.0,) * dim, (1.0,) * dim, r, r, f"uniform{dim}d_{n}")


def tall(nrows, n, seed):
    """A 2D grid of 3 x nrows cells."""
    rng = np.random.default_rng(seed)
    pos = rng.uniform(0, 1, size=(n, 2)) * (2.999, nrows - 0.001)
    return W.ParticleSet(pos, (0.0, 0.0), (2.9995, nrows - 0.0005), 1.0, 1.0, f"tall_{nrows}")


def check(pss, rps, cols):
    for ps, rp, col in zip(pss, rps, cols):
        want = oracle.search_ps(ps) if ps.n else (np.zeros(1, np.int64), np.zeros(0, np.int32), None)
        np.testing.assert_array_equal(rp.cpu().numpy(), want[0], err_msg=ps.name)
        np.testing.assert_array_equal(col.cpu().numpy()[:want[0][-1]], want[1], err_msg=ps.name)


def args_of(pss):
    return [(torch.from_numpy(np.ascontiguousarray(p.pos)).cuda(), p.lo, p.hi, p.cell_size, p.radius) for p in pss]


SETS = {
    "fifty_nine": list(range(1, 60)), "sixty": list(range(0, 60)),
    "tiles_inside": [0, 1, 4095, 0, 4096, 4097, 3, 0],
    "many_tiles": [5, 70001, 0, 4096, 1],
    "one_4095": [4095], "one_4096": [4096], "one_65536": [65536], "one_65537": [65537], "none": [0], "none_twice": [0, 0],
}


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("name", SETS)
def test_row_pointers_of_sets(ctx, name, shift):
    pss = [uniform(n, 2, 7 + i) for i, n in enumerate(SETS[name])]
    print(f"[gpu] row pointers {name} shift={shift}", flush=True)
    cells = ctx.cells()
    cells.batch_build(args_of(pss))
    rps = [torch.full((p.n + 1 + shift,), -7, dtype=torch.int64, device="cuda")[shift:] for p in pss]
    nnz = cells.batch_count(rps)
    cols = [torch.zeros(k, dtype=torch.int32, device="cuda") for k in nnz]
    cells.batch_fill(rps, cols, [torch.zeros(k, dtype=torch.float32, device="cuda") for k in nnz])
    torch.cuda.synchronize()
    assert nnz == [int(r[-1]) for r in rps]
    check(pss, rps, cols)
    assert cells.batch_nnz() == nnz
    cells.batch_nnz_enqueue()
    assert cells.batch_nnz_fetch() == nnz
    cells.close()


def test_row_pointers_past_the_folded_scan(ctx):
    """More than 1024 tiles: a lattice without jitter, radius 1.2 spacings (4, 3 or 2 neighbours)."""
    side = 2100
    a = uniform(5, 2, 1)
    ij = np.stack(np.meshgrid(np.arange(side), np.arange(side), indexing="ij"), -1).reshape(-1, 2)
    lat = W.ParticleSet((ij + 0.5) / side, (0.0, 0.0), (1.0, 1.0), 1.2 / side, 1.2 / side, "lattice_2100")
    cells = ctx.cells()
    cells.batch_build(args_of([a, lat]))
    rps = [torch.empty(p.n + 1, dtype=torch.int64, device="cuda") for p in (a, lat)]
    nnz = cells.batch_count(rps)
    on = ((ij == 0) | (ij == side - 1)).sum(1)
    want = np.concatenate([[0], np.cumsum(4 - on)])
    np.testing.assert_array_equal(rps[1].cpu().numpy(), want)
    assert nnz[1] == want[-1]
    np.testing.assert_array_equal(rps[0].cpu().numpy(), oracle.search_ps(a)[0])
    cells.close()


@pytest.mark.parametrize("nrows", [8191, 8192, 8193, 8197])
def test_row_segments(ctx, nrows):
    ps = tall(nrows, 30000, nrows)
    print(f"[gpu] row segments {nrows}", flush=True)
    rp, col, _, _ = nnps.search(torch.from_numpy(ps.pos).cuda(), ps.lo, ps.hi, ps.cell_size, ps.radius, ctx=ctx)
    check([ps], [rp], [col])


@pytest.mark.parametrize("thresh", [-1, 40, 90])
@pytest.mark.parametrize("dim", [2, 3])
def test_blocks_of_uneven_rows(ctx, dim, thresh):
    """Cells of 0 to 200 particles along rows of more than two segments, with and without dense cells among them."""
    rng = np.random.default_rng(dim)
    ncx, ny = 150, 5
    occ = rng.choice([0, 0, 1, 2, 5, 30, 63, 64, 65, 128, 200], p=[.25, .25, .1, .1, .1, .1, .02, .02, .02, .02, .02],
                     size=ncx * ny)
    cell = np.repeat(np.arange(ncx * ny), occ)
    pos = np.zeros((cell.size, dim))
    pos[:, 0], pos[:, 1] = cell % ncx, cell // ncx
    pos += rng.uniform(0.01, 0.99, size=pos.shape)
    hi = (ncx - 0.001, ny - 0.001) + (0.999,) * (dim - 2)
    ps = W.ParticleSet(np.minimum(pos, np.asarray(hi))[rng.permutation(cell.size)], (0.0,) * dim, hi, 1.0, 0.5, f"uneven{dim}d")
    ctx.set_tuning(dense_min_union=thresh)
    cells = ctx.cells()
    for rep in range(2):
        print(f"[gpu] uneven rows {dim}d thresh={thresh} n={ps.n} rep={rep}", flush=True)
        rp, col, _, _ = nnps.search(torch.from_numpy(ps.pos).cuda(), ps.lo, ps.hi, ps.cell_size, ps.radius, ctx=ctx, cells=cells)
        check([ps], [rp], [col])
    cells.close()
    ctx.set_tuning()


@pytest.mark.parametrize("thresh", [-1, 1])
def test_counts_and_fills_repeat(ctx, thresh):
    """Long rows (thresh -1) or dense cells (1): a second count, a second and a third fill."""
    rng = np.random.default_rng(3)
    pos = np.concatenate([rng.uniform(0, 1, size=(4000, 3)), 0.5 + 0.02 * rng.standard_normal((3000, 3))])
    ps = W.ParticleSet(pos, (0.0,) * 3, (1.0,) * 3, 0.05, 0.05, "clump")
    ctx.set_tuning(dense_min_union=thresh)
    print(f"[gpu] repeats thresh={thresh}", flush=True)
    cells = ctx.cells()
    cells.batch_build(args_of([ps]))
    for count in range(2):
        rps = [torch.empty(ps.n + 1, dtype=torch.int64, device="cuda")]
        nnz = cells.batch_count(rps)
        for fill in range(2 + count):
            cols = [torch.zeros(nnz[0], dtype=torch.int32, device="cuda")]
            cells.batch_fill(rps, cols, [torch.zeros(nnz[0], dtype=torch.float32, device="cuda")])
            check([ps], rps, cols)
            st = cells.stats()
            assert (st["heavy_rows"] > 0) == (thresh < 0)
    cells.close()
    ctx.set_tuning()


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 1024, 1025, 2049, 5000])
@pytest.mark.parametrize("shape", ["one_cell", "own_cells", "shuffled_runs"])
def test_assignment_with_and_without_the_table(ctx, shape, n):
    """Slots taken through a workgroup's table (a first build, which expects dense cells) and run by
    run (the builds after a count that saw none): all particles in one cell, each in its own
    (more cells than half a table holds of one workgroup's), and short runs in random order."""
    rng = np.random.default_rng(n)
    side = 71
    if shape == "one_cell":
        cell = np.full(n, side * 30 + 40)
    elif shape == "own_cells":
        cell = rng.permutation(side * side)[:n]
    else:
        cell = rng.permutation(np.repeat(rng.integers(0, side * side, size=n // 3 + 1), 3)[:n].reshape(-1, 1)).ravel()
    pos = np.stack([cell % side, cell // side], 1) + rng.uniform(0.05, 0.95, size=(n, 2))
    ps = W.ParticleSet(pos, (0.0, 0.0), (side - 0.001,) * 2, 1.0, 0.05, f"{shape}_{n}")
    print(f"[gpu] assignment {shape} n={n}", flush=True)
    ctx.set_tuning(dense_min_union=100000)  # looked for, never seen
    cells = ctx.cells()
    for rep in range(2):
        rp, col, _, _ = nnps.search(torch.from_numpy(ps.pos).cuda(), ps.lo, ps.hi, ps.cell_size, ps.radius, ctx=ctx, cells=cells)
        check([ps], [rp], [col])
        assert cells.stats()["dense_rows"] == 0
    cells.close()
    ctx.set_tuning()
