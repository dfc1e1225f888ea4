"""Lists of cells with more bins than atoms: a cluster or a gas in a wide cell,
many small cells.  The list build then starts from the atoms, not from the bins.
Against a float64 brute force over all pairs, with single bins of more atoms
than a wavefront has lanes and more candidates than its table holds; in MD,
where the same build runs behind a gate, against an evaluation of the state;
and its cost, which must not grow with the empty bins."""
import time

import numpy as np
import pytest

from paper_2607_06969_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _system(pos, cell, seed, pbc=(1, 1, 1)):
    rng = np.random.default_rng(seed)
    pos = np.asarray(pos).astype(np.float32).astype(np.float64)
    return W.System(pos, rng.integers(0, 3, len(pos)).astype(np.int32), np.eye(3)[None] * cell,
                    np.array([0, len(pos)], dtype=np.int64), {}, np.array([pbc], dtype=np.int32))


def _gas(n, cell, seed):
    return _system(np.random.default_rng(seed).random((n, 3)) * cell * 0.9999, cell, seed)


def _clump(n, a, cell, seed, pbc=(1, 1, 1)):
    """n^3 sites of spacing a around a corner of the cell (through all its faces where they are periodic)."""
    rng = np.random.default_rng(seed)
    g = (np.arange(n) - n / 2) * a
    pos = np.stack(np.meshgrid(g, g, g, indexing="ij"), axis=-1).reshape(-1, 3) + rng.uniform(-0.1, 0.1, (n ** 3, 3))
    return _system(pos % cell if all(pbc) else pos + cell / 3, cell, seed, pbc)


SYSTEMS = {
    "gas_small": lambda: _gas(200, 60.0, 1),
    "gas": lambda: _gas(3000, 190.0, 2),
    "cluster": lambda: _clump(13, 2.0, 144.0, 3),
    "cluster_open": lambda: _clump(13, 2.0, 144.0, 4, (0, 1, 0)),
    # some 125 atoms in a bin
    "clump": lambda: _clump(6, 1.2, 90.0, 5),
    # 27 bins of some 110 atoms: more candidates than the table holds
    "searched": lambda: _clump(15, 1.25, 200.0, 6),
    # no more bins than slots, but all atoms in a fifth of them: another path once the first lists are known
    "cluster_near": lambda: _clump(13, 1.9, 60.0, 11),
    "many": lambda: W.concat_systems([_clump(2, 2.6, 24.0, 10 + c, (0, 0, 0)) for c in range(300)]),
}


@pytest.mark.parametrize("name", sorted(SYSTEMS))
def test_lists_match_bruteforce(name):
    from paper_2607_06969_amd import nep
    s = SYSTEMS[name]()
    hp = W.hp_gst()
    m = nep.NepModel(hp, W.random_params(hp, 1))
    b = nep.Batch.from_system(s)
    bins = s.n_cfg * 64 * (int(s.cells[0, 0, 0] / 24.1) + 1) ** 3
    assert 4 * (s.n_atoms + 192) < bins or name == "cluster_near"
    cap = 640
    lists = {w: [t.cpu().numpy() for t in m.neighbors(b, w, cap=cap)] for w in (0, 1, 2, 3)}
    for c in range(s.n_cfg):
        a0, e0 = int(s.atom_off[c]), int(s.atom_off[c + 1])
        x, L, per = s.pos[a0:e0], np.diag(s.cells[c]), s.pbc_array()[c]
        d2 = np.zeros((e0 - a0,) * 2)
        for k in range(3):
            r = x[None, :, k] - x[:, None, k]
            d2 += (r - np.round(r / L[k]) * L[k] * per[k]) ** 2
        np.fill_diagonal(d2, np.inf)
        for which, rc in ((0, 6.0), (1, 4.0), (2, 4.0)):
            cnt, nb, _ = lists[which]
            for i in range(e0 - a0):
                k = int(cnt[a0 + i])
                got = nb[a0 + i, :k] - a0
                # pairs within 1e-4 A of the cutoff may fall on either side in float32
                sure = np.flatnonzero(d2[i] < (rc - 1e-4) ** 2)
                assert k <= cap and len(np.unique(got)) == k and np.isin(sure, got).all()
                assert (d2[i, got] < (rc + 1e-4) ** 2).all()
                assert np.all(np.diff(s.species[a0 + got]) >= 0)
    cnt, nb, _ = lists[2]
    cn3, rev, _ = lists[3]
    assert np.array_equal(cnt, cn3)
    for i in range(s.n_atoms):
        j, r = nb[i, :cnt[i]], rev[i, :cnt[i]]
        assert (r >= 0).all() and (r < cnt[j]).all() and (nb[j, r] == i).all()


LARGE = {"gas": lambda: _gas(70000, 400.0, 20), "cluster": lambda: _clump(41, 2.0, 400.0, 21),
         "cluster_open": lambda: _clump(41, 2.0, 400.0, 22, (1, 0, 0))}


@pytest.mark.parametrize("name", sorted(LARGE))
def test_large_lists_match_tree(name):
    """Beyond 49,152 slots, where a thread takes an atom: the pairs of a k-d tree (its periodic images as atoms of
    their own) as a sorted list."""
    from scipy.spatial import cKDTree

    from paper_2607_06969_amd import nep
    s = LARGE[name]()
    hp = W.hp_gst()
    b = nep.Batch.from_system(s)
    m = nep.NepModel(hp, W.random_params(hp, 1))
    L, per, n = s.cells[0, 0, 0], s.pbc_array()[0], s.n_atoms
    x, src = s.pos, np.arange(n)
    for k in range(3):
        if per[k]:
            lo, hi = x[:, k] < 6.1, x[:, k] > L - 6.1
            up, dn = x[lo].copy(), x[hi].copy()
            up[:, k] += L
            dn[:, k] -= L
            x, src = np.concatenate([x, up, dn]), np.concatenate([src, src[lo], src[hi]])
    pairs = cKDTree(x).query_pairs(6.0002, output_type="ndarray")
    pairs = np.concatenate([pairs, pairs[:, ::-1]])
    pairs = pairs[pairs[:, 0] < n]
    d = np.linalg.norm(x[pairs[:, 1]] - x[pairs[:, 0]], axis=1)
    pair_id = pairs[:, 0] * n + src[pairs[:, 1]]
    cap = 160
    for which, rc in ((0, 6.0), (1, 4.0), (2, 4.0)):
        cnt, nb, _ = (t.cpu().numpy() for t in m.neighbors(b, which, cap=cap))
        assert cnt.max() <= cap
        mine = np.arange(cap)[None] < cnt[:, None]
        got = np.sort(np.repeat(np.arange(n), cnt) * n + nb[mine])
        # pairs within 1e-4 A of the cutoff may fall on either side in float32
        sure, maybe = np.sort(pair_id[d < rc - 1e-4]), pair_id[d < rc + 1e-4]
        assert len(np.unique(got)) == len(got) and np.isin(sure, got).all() and np.isin(got, maybe).all()
        spc = np.where(mine, s.species[np.where(mine, nb, 0)], 9)
        assert (np.diff(spc, axis=1) >= 0).all()
    cnt, nb, _ = (t.cpu().numpy() for t in m.neighbors(b, 2, cap=64))
    cn3, rev, _ = (t.cpu().numpy() for t in m.neighbors(b, 3, cap=64))
    mine = np.arange(64)[None] < cnt[:, None]
    i, j, r = np.nonzero(mine)[0], nb[mine], rev[mine]
    assert cnt.max() <= 64 and np.array_equal(cnt, cn3) and (r >= 0).all() and (nb[j, r] == i).all()


def _islands(n_side, atoms, gap, seed):
    """n_side^3 islands of `atoms` atoms, gap apart, every pair of an island within 4 A."""
    rng = np.random.default_rng(seed)
    g = np.stack(np.meshgrid(*[np.arange(-1, 2)] * 3, indexing="ij"), axis=-1).reshape(-1, 3)
    g = g[np.argsort((g ** 2).sum(-1), kind="stable")][:atoms] * 1.1
    at = np.stack(np.meshgrid(*[np.arange(n_side)] * 3, indexing="ij"), axis=-1).reshape(-1, 1, 3) * gap + gap / 2
    return _system((at + g[None] + rng.uniform(-0.05, 0.05, (n_side ** 3, atoms, 3))).reshape(-1, 3), n_side * gap, seed)


@pytest.mark.parametrize("n_side", [6, 15])
@pytest.mark.parametrize("atoms", [16, 17, 18])
def test_lists_as_long_as_their_capacity(n_side, atoms):
    """A fresh handle's lists of a thin gas hold 16 entries: islands of 17 atoms fill them to the last."""
    from paper_2607_06969_amd import nep
    s = _islands(n_side, atoms, 30.0, 30)
    hp = W.hp_gst()
    m = nep.NepModel(hp, W.random_params(hp, 1))
    b = nep.Batch.from_system(s)
    cnt, rev = (m.neighbors(b, 3, cap=32)[k].cpu().numpy() for k in (0, 1))
    nb = m.neighbors(b, 2, cap=32)[1].cpu().numpy()
    assert (cnt == atoms - 1).all()
    i, a = np.nonzero(np.arange(32)[None] < cnt[:, None])
    assert (nb[i, a] // atoms == i // atoms).all() and (rev[i, a] >= 0).all() and (nb[nb[i, a], rev[i, a]] == i).all()


@pytest.mark.parametrize("s", [lambda: _clump(12, 2.9, 150.0, 7), lambda: _gas(20000, 300.0, 8),
                               lambda: _gas(70000, 500.0, 9)], ids=["cluster", "gas", "gas_large"])
def test_md_rebuilds(s):
    """A gas has more slots than a gated launch has blocks, or takes a thread per atom.  Skin 0.3 A: several rebuilds in 40 steps."""
    from paper_2607_06969_amd import nep
    s = s()
    hp = W.hp_gst()
    m = nep.NepModel(hp, W.random_params(hp, 2, std=0.02))
    m.set_variants(0, 0)
    b = nep.Batch.from_system(s)
    v = torch.as_tensor(W.maxwell_boltzmann(s.species, W.MASSES_GST, 3000.0), dtype=torch.float32, device="cuda")
    md = nep.NepMD(m, b, v.contiguous(), W.MASSES_GST, 1.0, 0.3)
    md.step(40)
    st = md.state()
    assert md.stats()["rebuilds"] >= 4
    now = m.compute(nep.Batch(st["pos"].contiguous(), b.species, b.atom_off, b.cells, b.pbc))
    scale = float(now["F"].abs().max())
    # the positions of the state are rounded to float32 here and carried in float64 there: 1e-5 A at 300 A
    assert scale > 0 and float((now["F"] - st["F"]).abs().max()) < 1e-3 * scale


def _median_us(call, n=30):
    ts = []
    for _ in range(n):
        t0 = time.perf_counter()
        call()
        torch.cuda.synchronize()
        ts.append(time.perf_counter() - t0)
    return 1e6 * sorted(ts)[n // 3]


def test_cost_of_empty_bins():
    """1,000 atoms in a 1,000 A cell: 4.7 million bins.  What grows with them is the sort's passes over their
    counts, some 0.2 ms; a wavefront for each costs 1.1 ms more."""
    from paper_2607_06969_amd import nep
    hp = W.hp_gst()
    m = nep.NepModel(hp, W.random_params(hp, 3))
    b = nep.Batch.from_system(_gas(1000, 1000.0, 9))
    assert _median_us(lambda: m.descriptors(b)) < 700


def test_cost_of_lists_beyond_their_capacity():
    """900 open cells whose every list exceeds the capacity that the mean density suggests, on the workspace that
    starts from it in every call: two list builds (some 0.05 ms each), an atomic per wavefront on one word 0.8 ms more."""
    from paper_2607_06969_amd import nep
    hp = W.hp_gst()
    m = nep.NepModel(hp, W.random_params(hp, 3))
    s = W.concat_systems([_islands(1, 20, 40.0, 40 + c) for c in range(900)])
    s.pbc[:] = 0
    b = nep.Batch.from_system(s)
    kept, fresh = _median_us(lambda: m.compute(b)), _median_us(lambda: m.compute(b, noalloc=True))
    assert fresh < kept + 250


def test_cost_of_uneven_bins():
    """13,824 atoms 1.9 A apart in a 120 A cell: fewer bins than slots, but the full ones hold far more than the mean.
    0.19 ms; with every candidate searched for, a wavefront per full bin, 0.67."""
    from paper_2607_06969_amd import nep
    hp = W.hp_gst()
    m = nep.NepModel(hp, W.random_params(hp, 3))
    b = nep.Batch.from_system(_clump(24, 1.9, 120.0, 12))
    assert _median_us(lambda: m.descriptors(b)) < 400
