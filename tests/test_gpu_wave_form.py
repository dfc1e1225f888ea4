"""Variant 0 gives a wavefront to each atom in small batches and a thread in
large ones: both forms must agree bit for bit.  Variants 8 and 4 are the
one-thread form of variant 0 in other block sizes, at any batch size.  Systems
where the wavefront form changes its path: no neighbours at all, lists longer
than one round of 64, more angular pairs than a chunk of 32 holds, non-periodic
faces; and one configuration alone against itself inside a large batch."""
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


MODELS = {"small": W.hp_small_single, "gst": W.hp_gst, "table2": W.hp_table2}
SYSTEMS = {
    # about 185 (293) radial and 54 (106) angular neighbours: several rounds and chunks
    "dense": lambda t: _lattice(9, 1.7, 1, t),
    # between 33 and 64 angular neighbours for the longer cutoff only
    "medium": lambda t: _lattice(7, 2.3, 2, t),
    "slab_and_alone": lambda t: W.concat_systems([_lattice(6, 2.9, 3, t, [1, 1, 0]), _alone(t), _lattice(6, 3.1, 4, t)]),
}


def _everything(m, b, d, f):
    m.set_variants(d, f)
    out = m.compute(b, atom_energy=True, atom_virial=True)
    out["q"] = m.descriptors(b)
    n = b.n_atoms
    lab = [torch.linspace(-1, 1, b.n_cfg, dtype=torch.float64, device="cuda"),
           torch.linspace(-1, 1, 3 * n, device="cuda").view(n, 3).contiguous(),
           torch.linspace(-1, 1, 9 * b.n_cfg, dtype=torch.float64, device="cuda").view(-1, 9).contiguous()]
    out["loss"], out["grad"] = m.loss_grad(b, *lab)
    return out


@pytest.mark.parametrize("model", sorted(MODELS))
@pytest.mark.parametrize("system", sorted(SYSTEMS))
def test_wave_form_is_the_thread_form(model, system):
    from paper_2607_06969_amd import nep
    hp = MODELS[model]()
    m = nep.NepModel(hp, W.random_params(hp, 11))
    b = nep.Batch.from_system(SYSTEMS[system](hp.n_species))
    one, two = _everything(m, b, 0, 0), _everything(m, b, 8, 4)
    for k in one:
        assert torch.isfinite(one[k]).all(), k
        assert torch.equal(one[k], two[k]), k


def test_alone_equals_inside_a_large_batch():
    """The batch of 27,000 atoms runs one thread per atom, its parts alone one wavefront per atom."""
    from paper_2607_06969_amd import nep
    hp = W.hp_gst()
    m = nep.NepModel(hp, W.random_params(hp, 12))
    parts = [W.rocksalt_gst(8, seed=21), W.rocksalt_gst(30, seed=22), W.rocksalt_gst(14, seed=23)]
    s = W.concat_systems(parts)
    full = m.compute(nep.Batch.from_system(s))
    for c in (0, 2):
        one = m.compute(nep.Batch.from_system(s.config(c)))
        a, e = int(s.atom_off[c]), int(s.atom_off[c + 1])
        assert torch.equal(one["F"], full["F"][a:e])
        assert torch.equal(one["E"], full["E"][c:c + 1]) and torch.equal(one["V"], full["V"][c:c + 1])
