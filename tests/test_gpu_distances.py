"""The FP32 distances of the FP16 RCLL mode against binary64, in u = 2^-24: unbiased, and within
the sum of their roundings. Per axis the displacement errs by at most 1.25 quanta (two rounded
positions) and is rounded to FP32 (u); squares and sums add three roundings to the squared
distance at most, the root 1.02 u, and a power of two scales it: (2 + 3) / 2 + 1.02 u beside the
quanta, which at the smallest distance taken this way (sqrt(3) 2^23 quanta) are 2.5 u. Every
step rounds to nearest, so that the mean signed error of many pairs is near 0 (0.05 u allowed:
over these sets' 1e5 to 7e6 pairs of about 0.5 u each the mean of independent errors is below
0.002 u)."""
import numpy as np
import pytest

from paper_2401_08586_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2401_08586_amd import nnps  # noqa: E402

SETS = {"lattice2d": lambda: W.lattice(2, 200, 1.0 / 200, 0.1, seed=1),
        "lattice3d": lambda: W.lattice(3, 50, 1.0 / 50, 0.1, seed=2),
        "uniform2d": lambda: W.uniform(2, 60000, seed=3),
        "uniform3d": lambda: W.uniform(3, 60000, seed=4)}


@pytest.mark.parametrize("dense", [False, True], ids=["blocks", "dense"])
@pytest.mark.parametrize("name", SETS)
def test_distances_are_unbiased(name, dense):
    ps = SETS[name]()
    print(f"[gpu] distances {name} dense={dense}", flush=True)
    pos = torch.from_numpy(ps.pos).cuda()
    ctx = nnps.Context(0)
    try:
        ctx.set_tuning(dense_min_union=1 if dense else -1)
        cells = ctx.cells()
        for _ in range(2):  # dense cells: tested in the fill, then taken from the count's bits
            rp, col, dist, _ = nnps.search(pos, ps.lo, ps.hi, ps.cell_size, ps.radius, mode=nnps.MODE_FP16_RCLL, ctx=ctx,
                                           cells=cells)
            rows = torch.repeat_interleave(torch.arange(ps.n, device="cuda"), rp[1:] - rp[:-1])
            d = pos[col.long()] - pos[rows]
            want = torch.sqrt((d * d).sum(1))
            err = ((dist.double() - want) / want).cpu().numpy() * 2.0 ** 24
            print(f"  mean {np.abs(err).mean():.4f} max {np.abs(err).max():.3f} bias {err.mean():+.4f} of {err.size}", flush=True)
            assert abs(err.mean()) <= 0.05
            assert np.abs(err).max() <= 2.5 + 1.02 + 2.5
        cells.close()
    finally:
        ctx.set_tuning()
        ctx.close()


@pytest.mark.parametrize("mode", [nnps.MODE_FP16_RCLL, nnps.MODE_RECHECK_ALL])
@pytest.mark.parametrize("name", SETS)
def test_distances_are_the_same_on_every_path(name, mode):
    """Bit for bit in blocks, in dense cells tested by the fill, in dense cells from the count's bits
    and (unions past the block limit) in long rows; recheck-all's are the FP16 mode's."""
    ps = SETS[name]()
    far = W.ParticleSet(ps.pos, ps.lo, ps.hi, 4 * ps.cell_size, ps.radius)  # wide cells: large unions
    pos = torch.from_numpy(ps.pos).cuda()
    ctx = nnps.Context(0)
    try:
        for p in (ps, far):
            first = None
            for m, dense in ((nnps.MODE_FP16_RCLL, -1), (mode, -1), (mode, 1)):
                print(f"[gpu] paths {name} cell={p.cell_size} mode={m} dense={dense}", flush=True)
                ctx.set_tuning(dense_min_union=dense)
                cells = ctx.cells()
                for _ in range(2):
                    dist = nnps.search(pos, p.lo, p.hi, p.cell_size, p.radius, mode=m, ctx=ctx, cells=cells)[2]
                    first = dist if first is None else first
                    assert torch.equal(dist.view(torch.int32), first.view(torch.int32))
                cells.close()
    finally:
        ctx.set_tuning()
        ctx.close()
