"""The float64 evaluation gives small batches a wavefront per atom: against the
FP64 oracle where it changes its path (lists of several rounds, more angular pairs
than a chunk of 16, no pairs, padding beside an atom, a species without atoms), and
on both sides of its size limit against the configurations alone.

Tolerances: those of the existing comparisons, 1e-10; two results 2e-10."""
import numpy as np
import pytest

from paper_2607_06969_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _lattice(n, a, seed, species, pbc=None):
    s = W.simple_cubic(n=n, spacing=a, sigma=0.08, seed=seed, species_count=species)
    s.pbc = None if pbc is None else np.array([pbc], dtype=np.int32)
    return s


def _alone(species):
    return W.System(np.array([[1.0, 2.0, 3.0]]), np.array([species - 1], dtype=np.int32), np.eye(3)[None] * 20.0,
                    np.array([0, 1], dtype=np.int64))


def _one_species(t):
    s = _lattice(6, 2.9, 6, t)
    s.species[:] = t - 1
    return s


MODELS = {"small": W.hp_small_single, "gst": W.hp_gst, "table2": W.hp_table2}
SYSTEMS = {
    "dense": lambda t: _lattice(9, 1.7, 1, t),
    "slab_and_alone": lambda t: W.concat_systems([_lattice(6, 2.9, 3, t, [1, 1, 0]), _alone(t), _lattice(6, 3.1, 4, t)]),
    "one_species_only": _one_species,
    "alone": _alone,
}


def _rel(a, b):
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)


def _compute(m, p, s):
    from paper_2607_06969_amd import nep
    out = m.compute64(nep.Batch.from_system(s), torch.tensor(p, dtype=torch.float64, device="cuda"), atom_energy=True)
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("model", sorted(MODELS))
@pytest.mark.parametrize("system", sorted(SYSTEMS))
def test_compute64_matches_oracle(oracle_lib, model, system):
    from paper_2607_06969_amd import nep
    hp = MODELS[model]()
    s = SYSTEMS[system](hp.n_species)
    p = W.random_params(hp, 21)
    print(f"[wave64] {model} {system} N={s.n_atoms}", flush=True)
    ref = oracle_lib.evaluate(hp, p, s, nbr_mode=2)
    got = _compute(nep.NepModel(hp, p), p, s)
    assert np.max(np.abs(got["E"] - ref["E"]) / np.diff(s.atom_off)) <= 1e-10
    assert _rel(got["F"], ref["F"]) <= 1e-10
    assert _rel(got["V"].reshape(-1, 9), ref["V"].reshape(-1, 9)) <= 1e-10


def test_both_sides_of_the_size_rule():
    from paper_2607_06969_amd import nep
    hp = W.hp_gst()
    p = W.random_params(hp, 22)
    m = nep.NepModel(hp, p)
    parts = [_lattice(n, 3.0, n, 3) for n in (30, 31)]  # 27,000 and 29,791 atoms
    both = W.concat_systems(parts)
    print(f"[wave64] N={both.n_atoms}", flush=True)
    full = _compute(m, p, both)
    for c, s in enumerate(parts):
        one = _compute(m, p, s)
        a, e = both.atom_off[c], both.atom_off[c + 1]
        assert abs(one["E"][0] - full["E"][c]) / s.n_atoms <= 2e-10
        assert _rel(full["F"][a:e], one["F"]) <= 2e-10 and _rel(full["Ei"][a:e], one["Ei"]) <= 2e-10
        assert _rel(full["V"].reshape(-1, 9)[c], one["V"].reshape(-1, 9)[0]) <= 2e-10
