"""Pairs across the face of a cell so long that float32 coordinates are some
0.01 A apart: the list holds every pair whose float32 pair vector, r_j - r_i plus
the lattice shift, lies within the cutoff, whatever the list build tests on the
way (it drops candidates by their distance from a box of atoms, rounded
otherwise).  The pairs here are those for which the two roundings differ most."""
import numpy as np
import pytest

from paper_2607_06969_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# the coordinates near the upper face have half the spacing of those beyond it
L = 131073.0
RC = 6.0


def _pairs(n):
    """x_i near 0, x_j near L and a difference in y: the float32 pair vector within the cutoff, position plus shift
    well beyond it."""
    f = np.float32
    rng = np.random.default_rng(3)
    xj = (131070.0 + rng.integers(0, 100, 400000) / 128.0).astype(f)
    xi = (5.5 - (L - xj.astype(np.float64)) + rng.uniform(-0.3, 0.3, len(xj))).astype(f)
    direct, image = (xi - xj) + f(L), (xi + f(L)) - xj
    take = np.argsort(direct - image, kind="stable")[:n]
    xi, xj, direct, image = xi[take], xj[take], direct[take], image[take]
    dy = np.sqrt(RC * RC - 1e-3 - direct.astype(np.float64) ** 2).astype(f)
    return xi, xj, dy, direct, image


def test_pairs_across_a_distant_face():
    from paper_2607_06969_amd import nep
    n = 40
    xi, xj, dy, direct, image = _pairs(n)
    pos = np.full((n, 2, 3), 4.0, dtype=np.float32)
    pos[:, 0, 0], pos[:, 1, 0] = xi, xj
    pos[:, 0, 1] += dy
    ry = (pos[:, 0, 1] - pos[:, 1, 1]).astype(np.float64)
    assert (direct.astype(np.float64) ** 2 + ry ** 2 < RC ** 2 - 1e-4).all()
    assert (image.astype(np.float64) ** 2 + ry ** 2 > (RC + 0.005) ** 2).all()
    pos = pos.astype(np.float64)
    s = W.System(pos.reshape(-1, 3), np.arange(2 * n, dtype=np.int32) % 3, np.repeat(np.diag([L, 20.0, 20.0])[None], n, 0),
                 np.arange(n + 1, dtype=np.int64) * 2)
    hp = W.hp_gst()
    m = nep.NepModel(hp, W.random_params(hp, 1))
    b = nep.Batch.from_system(s)
    cnt, nb, rv = (t.cpu().numpy() for t in m.neighbors(b, 0, cap=4))
    partner = np.arange(2 * n) ^ 1
    assert (cnt == 1).all(), f"{int((cnt != 1).sum())} of {2 * n} atoms without their neighbour"
    assert np.array_equal(nb[:, 0], partner)
    assert np.array_equal(rv[0::2, 0, 0], -direct) and np.array_equal(rv[1::2, 0, 0], direct)
