"""The statistics are those of the counted structure, whatever the caller's positions hold by the
time they are asked for, and recheck-all's comparison sees a wrong decision of the FP16 mode's
matrix test as well as of the packed FP16 test."""
import ctypes

import native_harness as native
import numpy as np
import pytest

from paper_2401_08586_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2401_08586_amd import nnps  # noqa: E402


@pytest.mark.parametrize("dense", [False, True], ids=["blocks", "dense"])
@pytest.mark.parametrize("mode", [nnps.MODE_FP16_RCLL, nnps.MODE_FP64_BASELINE, nnps.MODE_RECHECK_ALL,
                                  nnps.MODE_FP32_RCLL])
@pytest.mark.parametrize("dim", [2, 3])
def test_statistics_after_the_positions_changed(dim, mode, dense):
    ps = W.clustered(3000, 9, dim=dim)
    print(f"[gpu] statistics {dim}d mode={mode} dense={dense}", flush=True)
    pos = torch.from_numpy(ps.pos).cuda()
    ctx = nnps.Context(0)
    try:
        ctx.set_tuning(dense_min_union=1 if dense else -1)
        cells = ctx.cells()
        cells.build(pos, ps.lo, ps.hi, ps.cell_size, ps.radius, mode=mode)
        cells.count(torch.empty(ps.n + 1, dtype=torch.int64, device="cuda"))
        want = cells.stats()
        assert (want["dense_rows"] > 0) == dense
        pos.fill_(0.5)
        assert cells.stats() == want
        cells.close()
    finally:
        ctx.set_tuning()
        ctx.close()


@pytest.mark.parametrize("dense", [False, True], ids=["blocks", "dense"])
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("n", [2, 64, 150])
def test_recheck_all_sees_wrong_decisions(dim, n, dense):
    """Particles of one cell, three of them with the coordinate record of another place: every
    pair that this moves across the cutoff is counted once for the packed test and once for the
    matrix test. No pair, true or moved, is nearer to the cutoff than 0.03 squared cell widths,
    three times the wider test's band, so the decisions are known."""
    rng = np.random.default_rng(n + dim)
    radius, margin = 0.5, 0.03

    def clear(x, others):
        return np.all(np.abs(((others - x) ** 2).sum(1) - radius * radius) > margin)

    pos, rec = [], []
    while len(pos) < n:
        x = rng.uniform(0.02, 0.98, size=dim)
        y = rng.uniform(0.02, 0.98, size=dim) if len(pos) % 50 == 1 else x
        if not pos or (clear(x, np.array(pos)) and clear(y, np.array(rec)) and clear(x, np.array(rec)) and
                       clear(y, np.array(pos))):
            pos.append(x)
            rec.append(y)
        elif n > 2 and rng.random() < 0.01:  # a crowded corner: near points of an accepted one stay clear of the rest
            k = rng.integers(len(pos))
            pos.append(pos[k])
            rec.append(rec[k])
    pos, rec = np.array(pos), np.array(rec)

    def near(p):
        return ((p[:, None] - p[None]) ** 2).sum(-1) <= radius * radius

    want = int((near(pos) != near(rec)).sum())
    f16 = lambda x: np.float16(x)  # noqa: E731
    lo, hi, mid = 4 * (radius ** 2 - 2.0 ** -7), 4 * (radius ** 2 + 2.0 ** -7), 4 * radius ** 2
    t = [f16(lo), f16(hi), f16(mid)]
    assert all(float(a) == b for a, b in zip(t, (lo, hi, mid)))  # exact in FP16: no directed rounding here
    spos = np.zeros((n, 4))
    spos[:, :dim] = pos
    spos[:, 3] = np.arange(n, dtype=np.int64).view(np.float64)
    rq = np.zeros((n, 4), np.float32)
    rq[:, :dim] = 2 * rec - 1
    nb, nu = (n + 63) // 64, (n + 63) // 64
    arrays = dict(pos=pos, set_room=np.zeros(native.load().harness_set_bytes(), np.uint8), offs=np.array([0, n], np.int32),
                  cell_offs=np.array([0, 1], np.int32), skey=np.zeros(n, np.uint32), perm=np.arange(n, dtype=np.int32),
                  cell_start=np.array([0, n], np.int32), spos=spos, rq=rq, flags=np.zeros(8, np.int32),
                  bstart=np.minimum(64 * np.arange(nb + 1), n).astype(np.int32), bset=np.zeros(nb, np.int32),
                  nblk=np.array([0 if dense else nb], np.int32), blk_stats=np.zeros((nb, 5), np.uint64),
                  stats=np.zeros(16, np.uint64), wdense=np.ones(1, np.int32), usz=np.array([n], np.int32),
                  uoff=np.array([0, n], np.int64), ulist=np.arange(n, dtype=np.int32), unit_off=np.array([0, nu], np.int32),
                  ucell=np.zeros(nu, np.int32), dn=np.array([n], np.int32), dstats=np.zeros((2, 6), np.uint64))
    dev = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in arrays.items()}
    args = native.Args(dim=dim, mode=nnps.MODE_RECHECK_ALL, n=n, radius=radius, nblk_max=nb,
                       t_lo=int(t[0].view(np.uint16)), t_hi=int(t[1].view(np.uint16)), t_mid=int(t[2].view(np.uint16)))
    for k, v in dev.items():
        setattr(args, k, v.data_ptr())
    torch.cuda.synchronize()
    print(f"[gpu] wrong decisions {dim}d n={n} dense={dense} want={want}", flush=True)
    assert native.load().harness_stats(ctypes.byref(args), int(dense)) == 0
    assert n == 2 or want > 0
    assert int(dev["stats"].cpu().numpy()[4]) == 2 * want
