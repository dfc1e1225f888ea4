"""Energy and virial of every configuration are the float64 sums of the per-atom
values, summed in the launch of the force gather by one block per chunk: chunk
edges (one atom, 512, 513, several chunks, the sizes where the chunks grow),
every block size of the gather, and calls one after another (the counters that
find a configuration's last chunk are left clear).

Tolerance: float64 sums in two orders, n * 2^-52 of the sum of magnitudes."""
import numpy as np
import pytest

from paper_2607_06969_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _atoms(n, seed):
    """n atoms on a jittered lattice in a box with room for them."""
    k = max(6, int(np.ceil(n ** (1 / 3) - 1e-9)))
    s = W.simple_cubic(n=k, spacing=3.0, sigma=0.1, seed=seed, species_count=3)
    return W.System(s.pos[:n], s.species[:n], s.cells, np.array([0, n], dtype=np.int64))


BATCHES = {"edges": (1, 511, 512, 513, 2049, 3), "growth": (64000, 65537), "one": (700,)}


@pytest.mark.parametrize("gather", [0, 1, 2, 3])
@pytest.mark.parametrize("batch", sorted(BATCHES))
def test_sums_are_the_sums(batch, gather):
    from paper_2607_06969_amd import nep
    hp = W.hp_gst()
    p = W.random_params(hp, 5)
    s = W.concat_systems([_atoms(n, 40 + i) for i, n in enumerate(BATCHES[batch])])
    m = nep.NepModel(hp, p)
    m.set_gather_variant(gather)
    m.reuse_lists(True)
    b = nep.Batch.from_system(s)
    print(f"[sums] {batch} gather {gather} N={s.n_atoms}", flush=True)
    first = None
    for _ in range(3):
        out = {k: v.cpu().numpy() for k, v in m.compute(b, atom_energy=True, atom_virial=True).items()}
        for c in range(s.n_cfg):
            lo, hi = s.atom_off[c], s.atom_off[c + 1]
            for total, each in ((out["E"][c], out["Ei"]), (out["V"].reshape(-1, 9)[c], out["Wi"].reshape(-1, 9))):
                x = each[lo:hi].astype(np.float64)
                tol = (hi - lo) * 2.0 ** -52 * np.abs(x).sum(axis=0)
                assert np.all(np.abs(total - x.sum(axis=0)) <= tol), c
        if first is None:
            first = out
        for k in out:
            assert np.array_equal(out[k], first[k]), k
