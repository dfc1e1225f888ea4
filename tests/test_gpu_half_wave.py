"""At low mean densities the small-batch kernels give an atom half a wavefront:
bit for bit the one-thread kernels (variants 8 and 4), also where the two atoms of
a wavefront take different paths: lists of many rounds beside lonely atoms, more
angular pairs than a chunk of 16, padding beside an atom, an odd number of slots
at the end, several species."""
import numpy as np
import pytest

from paper_2607_06969_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MODELS = {"small": W.hp_small_single, "gst": W.hp_gst, "table2": W.hp_table2}


def _cluster(n, spacing, species, extra=0):
    """A lattice of n^3 atoms and `extra` lonely ones in a wide open box."""
    s = W.simple_cubic(n=n, spacing=spacing, sigma=0.08, seed=n, species_count=species)
    pos = np.concatenate([s.pos + 20.0, 5.0 + 8.0 * np.arange(extra)[:, None] * np.array([[1.0, 0.0, 0.0]])])
    spec = np.concatenate([s.species, np.arange(extra) % species]).astype(np.int32)
    order = np.random.default_rng(n).permutation(len(pos))
    return W.System(pos[order].astype(np.float32).astype(np.float64), spec[order], np.eye(3)[None] * 60.0,
                    np.array([0, len(pos)], dtype=np.int64), {}, np.zeros((1, 3), dtype=np.int32))


SYSTEMS = {
    "dense_cluster": lambda t: _cluster(8, 1.7, t, 5),   # up to some 290 radial, 100 angular pairs
    "cluster": lambda t: _cluster(7, 2.4, t, 1),         # around 16 angular pairs and more
    "few": lambda t: _cluster(2, 2.6, t, 1),
    "one": lambda t: _cluster(1, 3.0, t),
    "batch": lambda t: W.concat_systems([_cluster(3, 2.2, t, 3), _cluster(1, 3.0, t), _cluster(5, 2.7, t, 2)]),
}


@pytest.mark.parametrize("model", sorted(MODELS))
@pytest.mark.parametrize("system", sorted(SYSTEMS))
def test_half_wave_is_the_thread_form(model, system):
    from paper_2607_06969_amd import nep
    hp = MODELS[model]()
    s = SYSTEMS[system](hp.n_species)
    m = nep.NepModel(hp, W.random_params(hp, 12))
    b = nep.Batch.from_system(s)
    print(f"[half wave] {model} {system} N={s.n_atoms}", flush=True)
    out = []
    for d, f in ((0, 0), (8, 4)):
        m.set_variants(d, f)
        o = m.compute(b, atom_energy=True, atom_virial=True)
        o["q"] = m.descriptors(b)
        out.append(o)
    for k in out[0]:
        assert torch.isfinite(out[0][k]).all(), k
        assert torch.equal(out[0][k], out[1][k]), k


@pytest.mark.parametrize("large", [34, 38])
def test_alone_equals_inside_a_batch_on_both_sides_of_the_size_rule(large):
    """Batches of 35,300 and 49,300 sites (less the vacancies): lane groups, one
    thread per atom."""
    from paper_2607_06969_amd import nep
    hp = W.hp_gst()
    m = nep.NepModel(hp, W.random_params(hp, 12))
    s = W.concat_systems([W.rocksalt_gst(8, seed=21), W.rocksalt_gst(large, seed=22)])
    full = m.compute(nep.Batch.from_system(s))
    one = m.compute(nep.Batch.from_system(s.config(0)))
    assert torch.equal(one["F"], full["F"][:int(s.atom_off[1])])
    assert torch.equal(one["E"], full["E"][:1]) and torch.equal(one["V"], full["V"][:1])
