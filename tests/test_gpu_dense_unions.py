"""The dense cells' candidate lists where they are made differently: sets within one window of
indices (262,144), across two, at the last size that is ranked (four windows) and the first
that is sorted. A clump whose particles are numbered across the whole set, in a thin
background; the clump's rows against the CPU oracle, equal."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2401_08586_amd import nnps  # noqa: E402

WINDOW = 32 * 16 * 512


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("n", [3000, WINDOW - 1, WINDOW, WINDOW + 1, 2 * WINDOW + 1, 4 * WINDOW, 4 * WINDOW + 1])
def test_union_lists(dim, n):
    rng = np.random.default_rng(n)
    m = 2500
    at = np.unique(np.concatenate([np.linspace(0, n - 1, m - 4).astype(np.int64),
                                   [k for k in (WINDOW - 1, WINDOW, n - 2, n - 1) if k < n]]))
    pos = rng.uniform(0, 1, size=(n, dim))
    # the clump fills two cells a side, off the box's middle
    r = 0.5 * (1.0 / n) ** (1.0 / dim)
    pos[at] = 0.4 + 2.0 * r * rng.uniform(0, 1, size=(len(at), dim))
    ctx = nnps.Context(0)
    try:
        ctx.set_tuning(dense_min_union=200)
        print(f"[gpu] union lists {dim}d n={n}", flush=True)
        rp, col, _, cells = nnps.search(torch.from_numpy(pos).cuda(), (0.0,) * dim, (1.0,) * dim, r, r, ctx=ctx)
        assert cells.stats()["dense_rows"] > 0.5 * len(at)
        rp, col = rp.cpu().numpy(), col.cpu().numpy()
        rows = at[:: max(1, len(at) // 400)]
        wrp, wcol, _ = oracle.search_rows(pos, (0.0,) * dim, (1.0,) * dim, r, r, rows)
        for k, i in enumerate(rows):
            np.testing.assert_array_equal(col[rp[i]:rp[i + 1]], wcol[wrp[k]:wrp[k + 1]])
    finally:
        ctx.set_tuning()
        ctx.close()
