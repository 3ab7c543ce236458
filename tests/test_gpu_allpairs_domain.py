"""The all-list count of positions that are not finite: NNPS_EDOMAIN, and rows that still count
pairs: a particle that is no neighbour of itself (infinity or NaN) is not taken off its row."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2401_08586_amd import nnps  # noqa: E402


@pytest.mark.parametrize("n", [3, 200, 2500, 9000])
@pytest.mark.parametrize("dim", [2, 3])
def test_rows_of_positions_that_are_not_finite(dim, n):
    rng = np.random.default_rng(n)
    pos = rng.uniform(0, 1, size=(n, dim))
    bad = rng.choice(n, 3, replace=False)
    pos[bad[0], 0] = np.nan
    pos[bad[1], dim - 1] = np.inf
    pos[bad[2], 1] = -np.inf
    ok = np.delete(np.arange(n), bad)
    d2 = np.zeros(n, np.int64)
    for i in range(0, len(ok), 500):
        e = pos[ok][None] - pos[ok[i:i + 500]][:, None]
        d2[ok[i:i + 500]] = ((e * e).sum(-1) <= 0.25).sum(1) - 1
    want = np.concatenate([[0], np.cumsum(d2)])
    print(f"[gpu] all-list domain {dim}d n={n}", flush=True)
    ctx = nnps.Context(0)
    try:
        rp = torch.full((n + 1,), -5, dtype=torch.int64, device="cuda")
        col = torch.empty(1, dtype=torch.int32, device="cuda")
        dist = torch.empty(1, dtype=torch.float32, device="cuda")
        st, _ = nnps.allpairs_search_noalloc(torch.from_numpy(pos).cuda(), (0.0,) * dim, (1.0,) * dim, 0.5, rp, col, dist, ctx)
        assert st == nnps.NNPS_EDOMAIN
        np.testing.assert_array_equal(rp.cpu().numpy(), want)
    finally:
        ctx.close()
