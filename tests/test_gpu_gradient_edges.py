"""Rows that add nothing: exactly +0 in both gradients, also where the kernel's normalisation
(h^-3 in 2D, h^-4 in 3D) overflows, and a normalised gradient that does not depend on it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2401_08586_amd import nnps  # noqa: E402


@pytest.mark.parametrize("h", [1e-120, 1e-80, 1e-3, 1.0, 1e60])
@pytest.mark.parametrize("dim", [2, 3])
def test_rows_that_add_nothing(dim, h):
    """Row 0 empty, row 1 itself only, row 2 a coincident particle, row 3 one at 4h, row 4 one at h along
    the first axis: only the last adds."""
    pos = np.zeros((6, dim))
    pos[3, 0] = 4 * h
    pos[4, 0] = 8 * h
    pos[5, 0] = 9 * h
    f = np.array([1.0, 2.0, 3.0, 4.0, 5.0, 7.0])
    rp = np.array([0, 0, 1, 2, 3, 4, 4], np.int64)
    col = np.array([1, 0, 0, 5], np.int32)
    print(f"[gpu] gradient rows that add nothing {dim}d h={h}", flush=True)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    grad, norm = (t.cpu().numpy() for t in nnps.sph_gradient(up(pos), up(f), h, up(rp), up(col)))
    for g in (grad, norm):
        nothing = np.delete(g, 4, axis=0)
        assert np.all(nothing == 0) and not np.any(np.signbit(nothing))
    # (f_j - f_i) / (x_j - x_i) on the axis, within a few roundings; 0 off it
    assert abs(norm[4, 0] * h - 2.0) <= 2.0 * 16 * 2.0 ** -53 and np.all(norm[4, 1:] == 0)
