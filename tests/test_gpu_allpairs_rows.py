"""The all-list kernels at the sizes where they can go wrong: candidate steps of 64 (four of
them loaded together), workgroups of 4, 8 and 16 rows (the rows a wavefront takes change
after 2048 and 8192), the row scan's tiles of 4096, and one context's calls after one
another, a failing one among them. Against the CPU oracle, equal."""
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
    c.close()


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("n", [5, 63, 64, 65, 255, 256, 257, 2047, 2048, 2049, 4095, 4096, 4097, 8192, 8193])
def test_rows(ctx, dim, n):
    rng = np.random.default_rng(n)
    pos = rng.uniform(0, 1, size=(n, dim))
    r = 1.2 * (1.0 / n) ** (1.0 / dim)
    ps = W.ParticleSet(pos, (0.0,) * dim, (1.0,) * dim, r, r, f"rows{dim}d_{n}")
    print(f"[gpu] all-list rows {dim}d n={n}", flush=True)
    want = oracle.search_ps(ps)
    d = torch.from_numpy(pos).cuda()
    for rep in range(2):
        rp, col, dist = nnps.allpairs_search(d, ps.lo, ps.hi, ps.radius, ctx=ctx)
        np.testing.assert_array_equal(rp.cpu().numpy(), want[0])
        np.testing.assert_array_equal(col.cpu().numpy(), want[1])
        np.testing.assert_array_equal(dist.cpu().numpy().view(np.uint32), want[2].view(np.uint32))
        bad = d.clone()
        bad[n - 1, dim - 1] = float("nan") if rep else 1.5
        with pytest.raises(nnps.NnpsError) as e:
            nnps.allpairs_search(bad, ps.lo, ps.hi, ps.radius, ctx=ctx)
        assert e.value.code == nnps.NNPS_EDOMAIN
    assert ctx.check() == nnps.NNPS_OK
