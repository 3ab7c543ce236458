"""The dense count's kept bits where they cannot be kept: a cell with more than 2^31 (target, chunk)
pairs, on a structure that holds bits of an earlier search. Under the default bound they are not
asked for; under one above the device's memory the allocation fails and the search does without."""
import numpy as np
import pytest

import oracle
from paper_2401_08586_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2401_08586_amd import nnps  # noqa: E402


@pytest.mark.parametrize("bits_mib", [0, 1 << 20])
def test_more_pairs_than_32_bits(bits_mib):
    mode = nnps.MODE_FP16_RCLL
    n = 1600000  # in one cell: 1563 chunks, 2.5e9 pairs, 320 GB of bits
    ctx = nnps.Context(0)
    try:
        ctx.set_tuning(dense_bits_mib=bits_mib)
        cells = ctx.cells()
        ps = W.clustered(20000, 3, dim=3)
        small = torch.from_numpy(ps.pos).cuda()
        want = None
        for _ in range(2):  # the second keeps bits
            rp, col, dist, _ = nnps.search(small, ps.lo, ps.hi, ps.cell_size, ps.radius, mode=mode, ctx=ctx, cells=cells)
            assert cells.stats()["dense_rows"] > 0
            want = (rp, col, dist) if want is None else want
        pos = torch.rand(n, 3, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
        rp = torch.empty(n + 1, dtype=torch.int64, device="cuda")
        print(f"[gpu] dense bits n={n} bound={bits_mib}", flush=True)
        for _ in range(2):
            cells.build(pos, (0.0,) * 3, (1.0,) * 3, 2.0, 2.0, mode=mode)
            assert cells.count(rp) == n * (n - 1)  # all within the radius
            assert torch.equal(rp, torch.arange(n + 1, device="cuda") * (n - 1))
        got = nnps.search(small, ps.lo, ps.hi, ps.cell_size, ps.radius, mode=mode, ctx=ctx, cells=cells)
        assert all(torch.equal(a, b) for a, b in zip(got, want))
        cells.close()
    finally:
        ctx.set_tuning()
        ctx.close()


@pytest.mark.parametrize("mode", [nnps.MODE_FP16_RCLL, nnps.MODE_FP64_BASELINE])
@pytest.mark.parametrize("dim", [2, 3])
def test_lists_that_outgrow_the_kept_bits(dim, mode):
    """Updates contract a clustered set step by step, with no call that waits in between: the bits of
    the first steps fit the buffer, those of the last do not. Rows as the oracle's after every step."""
    ps = W.clustered(6000, 4, dim=dim)
    pos = torch.from_numpy(ps.pos.copy()).cuda()
    print(f"[gpu] outgrown bits {dim}d mode={mode}", flush=True)
    ctx = nnps.Context(0)
    try:
        cells = ctx.cells()
        rp = torch.empty(ps.n + 1, dtype=torch.int64, device="cuda")
        col = torch.empty(24_000_000, dtype=torch.int32, device="cuda")
        dist = torch.empty(24_000_000, dtype=torch.float32, device="cuda")
        for _ in range(2):
            cells.build(pos, ps.lo, ps.hi, ps.cell_size, ps.radius, mode=mode)
            cells.count(rp)
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        for step in range(6):
            d = -0.1 * (pos - 0.5)
            torch.cuda.synchronize()
            cells.batch_update_step([rp], [col], [dist], disp=[d], stream=stream)
            torch.cuda.synchronize()
            wrp, wcol, wdist = oracle.search_ps(W.ParticleSet(pos.cpu().numpy(), ps.lo, ps.hi, ps.cell_size, ps.radius))
            np.testing.assert_array_equal(rp.cpu().numpy(), wrp)
            np.testing.assert_array_equal(col[:len(wcol)].cpu().numpy(), wcol)
            got = dist[:len(wcol)].cpu().numpy().astype(np.float64)
            assert np.all(np.abs(got - wdist) <= 1e-6 * wdist)
        cells.close()
    finally:
        ctx.close()
