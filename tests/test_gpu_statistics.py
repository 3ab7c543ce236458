"""The statistics are those of the counted structure, whatever the caller's positions hold by the
time they are asked for."""
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
