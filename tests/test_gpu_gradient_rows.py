"""The gradient kernel at the row lengths where it can go wrong (0 to 33 entries: eight lanes
a row, two entries in flight a lane), with and without volumes, and its own square root and
reciprocal over pair distances from the smallest binary64 numbers to 1e150: one neighbour a
row, whose normalised gradient is exactly known up to rounding. Tolerances: the sum of a row
of m terms against the oracle's within the oracle's own bound for any order of summation;
single terms within 16 units in the last place (the term's dozen roundings)."""
import numpy as np
import pytest

from oracle import sph_gradient as G

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2401_08586_amd import nnps  # noqa: E402


@pytest.mark.parametrize("vol", [False, True])
@pytest.mark.parametrize("dim", [2, 3])
def test_row_lengths(dim, vol):
    rng = np.random.default_rng(dim)
    n = 3 * 34 + 5
    pos = rng.uniform(0, 1, size=(n, dim))
    f = rng.standard_normal(n)
    v = rng.uniform(0.5, 2.0, n) if vol else None
    lens = np.concatenate([np.repeat(np.arange(34), 3), [7, 0, 15, 16, 1]])
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = np.concatenate([rng.choice(np.delete(np.arange(n), i), size=m, replace=False) for i, m in enumerate(lens)])
    col = col.astype(np.int32)
    h = 0.9  # every pair inside 2h, on both sides of h
    print(f"[gpu] gradient row lengths {dim}d vol={vol}", flush=True)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    grad, norm = nnps.sph_gradient(up(pos), up(f), h, up(rp), up(col), vol=up(v) if vol else None)
    s, wnorm, (abs_s, abs_num, abs_den, num, den) = G.gradient(pos, f, h, rp, col, vol=v)
    # a term's own rounding beside the sum's: near q = 2 the factor (2 - q)^2 carries q's rounding
    d = np.concatenate([np.linalg.norm(pos[col[rp[i]:rp[i + 1]]] - pos[i], axis=1) for i in range(n) if lens[i]])
    assert np.all(np.abs(2 - d / h) > 0.05)
    assert np.all(np.abs(grad.cpu().numpy() - s) <= G.sum_bound(abs_s, lens + 40))
    bn, bd = G.sum_bound(abs_num, lens + 40), G.sum_bound(abs_den, lens + 40)
    nz = den != 0
    g = norm.cpu().numpy()
    assert np.all(g[~nz] == 0)
    tol = (bn[nz] + np.abs(wnorm[nz]) * bd[nz]) / (np.abs(den[nz]) - bd[nz]) * 1.01
    assert np.all(np.abs(g[nz] - wnorm[nz]) <= tol)


@pytest.mark.parametrize("scale", [5e-324, 1e-320, 1e-308, 1e-300, 1e-160, 1e-140, 1e-135, 1e-20, 1.0, 1e100, 1e135, 1e150])
def test_pair_distances(scale):
    """Particle 2k at 0 and 2k + 1 at x <= scale on one axis, each the other's only neighbour:
    grad = f_j dW/dr (x_i - x_j) / r, with r = |x| and the oracle's dW/dr."""
    x = np.array([1.0, 0.75, 0.5, 0.33, 1.0, 0.9]) * scale
    pos = np.zeros((12, 2))
    pos[1::2, 0] = x
    pos[7::2] = pos[7::2][:, ::-1]
    h = 0.8 * float(np.clip(scale, 1e-60, 1e100))  # h^-3 stays finite
    f = np.linspace(1.0, 2.0, 12)
    rp = np.arange(13, dtype=np.int64)
    col = (np.arange(12) ^ 1).astype(np.int32)
    print(f"[gpu] gradient pair distances {scale}", flush=True)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    grad, _ = nnps.sph_gradient(up(pos), up(f), h, up(rp), up(col))
    got = grad.cpu().numpy()
    for i in range(12):
        j = i ^ 1
        dx = pos[j] - pos[i]
        r2 = float(dx[0] * dx[0] + dx[1] * dx[1])  # as the kernel's: 0 when the squares underflow
        with np.errstate(over="ignore"):
            r = float(np.sqrt(r2))
        # (dx / r first: dW/dr / r alone underflows for the largest)
        want = np.zeros(2) if r == 0 or not np.isfinite(r) else -f[j] * G.kernel_dwdr(r, 2, h) * (dx / r)
        assert np.all(np.abs(got[i] - want) <= 16 * 2.0 ** -52 * np.abs(want) + 16 * 5e-324), (i, got[i], want)


def test_indices_outside_the_set_are_skipped():
    """An index outside [0, n) adds nothing, not even where the row's own field is infinite, and is reported."""
    ctx = nnps.Context(0)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    pos = np.array([[0.1, 0.1, 0.1], [0.2, 0.1, 0.1], [0.1, 0.25, 0.1]])
    f = np.array([np.inf, 2.0, 3.0])
    rp = np.array([0, 4, 6, 8], dtype=np.int64)
    col = np.array([1, 7, -1, 2, 2, 3, 1, -2147483648], dtype=np.int32)
    print("[gpu] gradient indices outside the set", flush=True)
    grad, _ = nnps.sph_gradient(up(pos), up(f), 0.2, up(rp), up(col), ctx=ctx)
    keep = (col >= 0) & (col < 3)
    crp = np.concatenate([[0], np.cumsum([keep[:4].sum(), keep[4:6].sum(), keep[6:].sum()])]).astype(np.int64)
    s, _, (abs_s, *_) = G.gradient(pos, np.where(np.isinf(f), 1.0, f), 0.2, crp, col[keep])
    assert np.all(np.abs(grad.cpu().numpy() - s) <= G.sum_bound(abs_s, np.full(3, 42)))
    assert ctx.check() == nnps.NNPS_EINVAL
    ctx.close()
