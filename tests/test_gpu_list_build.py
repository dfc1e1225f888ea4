"""The per-bin list build where its paths change: more than 64 kept entries
per atom (several rounds leave the stage), more than 64 atoms in a bin, more
candidates than its table holds, and bins split over several wavefronts.
Against a float64 brute force over all pairs."""
import numpy as np
import pytest

from paper_2607_06969_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _lattice(n, a, cell, pbc, seed):
    """n^3 sites of spacing a with a little disorder, three species, in a cubic cell of side `cell`."""
    rng = np.random.default_rng(seed)
    g = np.arange(n) * a + 0.5
    pos = np.stack(np.meshgrid(g, g, g, indexing="ij"), axis=-1).reshape(-1, 3) + rng.uniform(-0.1, 0.1, (n ** 3, 3))
    spc = rng.integers(0, 3, size=n ** 3).astype(np.int32)
    return W.System(pos.astype(np.float32).astype(np.float64), spc, np.eye(3)[None] * cell,
                    np.array([0, n ** 3], dtype=np.int64), {}, np.array([pbc], dtype=np.int32))


SYSTEMS = {
    # 8^3 sites at 2.2 A, periodic: about 85 neighbours within 6 A
    "dense": lambda: _lattice(8, 2.2, 17.6, [1, 1, 1], 1),
    # a cluster in a cell of one bin per direction: 216 atoms in one bin
    "one_bin": lambda: _lattice(6, 2.4, 7.0, [0, 0, 0], 2),
    # 13^3 = 2,197 atoms in one bin: more candidates than the table holds
    "searched": lambda: _lattice(13, 2.9, 8.0, [0, 0, 0], 3),
    # all of them, and one atom alone, in one batch
    "batch": lambda: W.concat_systems([_lattice(8, 2.2, 17.6, [1, 1, 1], 4), _lattice(1, 2.0, 30.0, [1, 1, 1], 5),
                                       _lattice(6, 2.4, 7.0, [0, 0, 0], 6), _lattice(9, 3.0, 27.0, [1, 1, 0], 7)]),
}


def _pairs(s, c, rc):
    sub = s.config(c)
    x, L, per = sub.pos, np.diag(sub.cells[0]), sub.pbc_array()[0]
    r = x[None, :, :] - x[:, None, :]
    r -= np.round(r / L) * L * per
    d = np.sqrt((r ** 2).sum(-1))
    np.fill_diagonal(d, np.inf)
    return d


@pytest.mark.parametrize("name", sorted(SYSTEMS))
@pytest.mark.parametrize("which,rc", [(0, 6.0), (1, 4.0), (2, 4.0)])
def test_lists_match_bruteforce(name, which, rc):
    from paper_2607_06969_amd import nep
    s = SYSTEMS[name]()
    hp = W.hp_gst()
    m = nep.NepModel(hp, W.random_params(hp, 1))
    cap = 160
    cnt, nb, _ = (t.cpu().numpy() for t in m.neighbors(nep.Batch.from_system(s), which, cap=cap))
    for c in range(s.n_cfg):
        a0 = int(s.atom_off[c])
        d = _pairs(s, c, rc)
        for i in range(len(d)):
            k = int(cnt[a0 + i])
            got = nb[a0 + i, :k] - a0
            assert k <= cap and len(set(got)) == k
            # pairs within 1e-4 A of the cutoff may fall on either side in float32
            sure, maybe = set(np.flatnonzero(d[i] < rc - 1e-4)), set(np.flatnonzero(d[i] < rc + 1e-4))
            assert sure <= set(got) <= maybe
            # rows are in processing order: the species never decrease
            assert np.all(np.diff(s.species[a0 + got]) >= 0)


@pytest.mark.parametrize("name", sorted(SYSTEMS))
def test_reverse_positions(name):
    """Every angular entry's partner entry points back (the lists are symmetric and whole)."""
    from paper_2607_06969_amd import nep
    s = SYSTEMS[name]()
    hp = W.hp_gst()
    m = nep.NepModel(hp, W.random_params(hp, 1))
    b = nep.Batch.from_system(s)
    cnt, nb, _ = (t.cpu().numpy() for t in m.neighbors(b, 2, cap=96))
    cn3, rev, _ = (t.cpu().numpy() for t in m.neighbors(b, 3, cap=96))
    assert np.array_equal(cnt, cn3) and cnt.max() <= 96
    for i in range(s.n_atoms):
        for a in range(cnt[i]):
            j, r = nb[i, a], rev[i, a]
            assert 0 <= r < cnt[j] and nb[j, r] == i and rev[j, r] == a
