"""Cells far from unit size: every mode finds the oracle's neighbours whatever the units, in
work blocks and in dense cells. (Radii above 2^100: the slots past a union's last candidate
were once put at a fixed squared distance of 2^200, which the binary64 tiles then took for
neighbours.)"""
import numpy as np
import pytest

import oracle
from paper_2401_08586_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2401_08586_amd import nnps  # noqa: E402

MODES = {"fp16": nnps.MODE_FP16_RCLL, "fp64": nnps.MODE_FP64_BASELINE, "fp32": nnps.MODE_FP32_RCLL,
         "recheck_all": nnps.MODE_RECHECK_ALL}


def blob(n, dim, seed, scale):
    """n points in the middle cell of a 5^dim grid, radius 0.7 cells."""
    pos = scale * (2.0 + np.random.default_rng(seed).uniform(0.02, 0.98, size=(n, dim)))
    return W.ParticleSet(pos, (0.0,) * dim, (5.0 * scale,) * dim, scale, 0.7 * scale, f"blob{dim}d_{n}_{scale:g}")


def sparse(dim, seed, scale):
    """About one point in eight cells of a grid of 64 cells along an axis: blocks span many cells."""
    n = 512 if dim == 2 else 32768
    pos = scale * 64.0 * np.random.default_rng(seed).uniform(0, 1, size=(n, dim))
    return W.ParticleSet(pos, (0.0,) * dim, (64.0 * scale,) * dim, scale, scale, f"sparse{dim}d_{scale:g}")


def straddle(dim, scale):
    """Row A: two targets 15.9 cells apart. Row B above it: 31 points near each of them in turn, those
    near the second its neighbours or just not, two of them 16.1 cells from the first target (their
    squares about it overflow at scale 2^508, the others' do not). 64 candidates: every sixteen of
    them hold some that are near either target."""
    near = np.stack([np.linspace(0.5, 0.9, 31), np.full(31, 1.2)], axis=1)
    far = np.stack([np.linspace(15.8, 16.0, 31), np.where(np.arange(31) % 2, 1.1, 1.48)], axis=1)
    far[20:22] = (16.6, 1.1), (16.6, 1.49)
    one = np.concatenate([[[0.5, 0.5], [16.4, 0.5]], np.stack([near, far], axis=1).reshape(-1, 2)])
    pos = (one[None] + np.array([0.0, 4.0]) * np.arange(5)[:, None, None]).reshape(-1, 2)
    if dim == 3:
        pos = np.concatenate([pos, np.full((len(pos), 1), 0.5)], axis=1)
    return W.ParticleSet(scale * pos, (0.0,) * dim, (64.0 * scale,) * dim, scale, scale, f"straddle{dim}d_{scale:g}")


def check(ps, mode, dense):
    print(f"[gpu] scales {ps.name} n={ps.n} {mode} dense={dense}", flush=True)
    wrp, wcol, wdist = oracle.search_ps(ps)
    ctx = nnps.Context(0)
    try:
        ctx.set_tuning(dense_min_union=1 if dense else -1)
        cells = ctx.cells()
        for _ in range(2):  # dense cells: tested in the fill, then taken from the count's bits
            rp, col, dist, _ = nnps.search(torch.from_numpy(ps.pos).cuda(), ps.lo, ps.hi, ps.cell_size, ps.radius,
                                           mode=MODES[mode], ctx=ctx, cells=cells)
            np.testing.assert_array_equal(rp.cpu().numpy(), wrp, err_msg=ps.name)
            np.testing.assert_array_equal(col.cpu().numpy(), wcol, err_msg=ps.name)
            d = dist.cpu().numpy()
            if mode in ("fp64", "fp32"):
                np.testing.assert_array_equal(d.view(np.uint32), wdist.view(np.uint32), err_msg=ps.name)
            else:
                # 1e-6 where FP32 has the distance (as a normal number), else the nearest it has
                w = wdist.astype(np.float64)
                normal = np.isfinite(wdist) & (w >= 2.0 ** -126)
                assert np.all(np.abs(d[normal].astype(np.float64) - w[normal]) <= 1e-6 * w[normal]), ps.name
                assert np.all(np.isinf(d[np.isinf(wdist)])), ps.name
        cells.close()
    finally:
        ctx.set_tuning()
        ctx.close()


@pytest.mark.parametrize("dense", [False, True], ids=["blocks", "dense"])
@pytest.mark.parametrize("mode", MODES)
def test_radius_above_2_to_100(mode, dense):
    for scale in (2e30, 1e36):
        for dim in (2, 3):
            for n in (2, 33, 200, 1025):
                check(blob(n, dim, n, scale), mode, dense)


@pytest.mark.parametrize("dense", [False, True], ids=["blocks", "dense"])
@pytest.mark.parametrize("mode", MODES)
def test_squares_at_the_ends_of_the_exponent_range(mode, dense):
    """Cells whose squared extent over a block overflows although every neighbour's squared
    distance is finite (from 2^506 on: a block's span of up to 64 cells is squared past 2^1024), and cells
    whose squares are subnormal or zero."""
    for e in (449, 451, 506, 507, 508, 510, -449, -451, -510, -520):
        check(sparse(3, e & 1023, 2.0 ** e), mode, dense)
        check(sparse(2, e & 1023, 2.0 ** e), mode, dense)
        check(blob(200, 3, e & 1023, 2.0 ** e), mode, dense)
        check(straddle(2, 2.0 ** e), mode, dense)
        check(straddle(3, 2.0 ** e), mode, dense)
