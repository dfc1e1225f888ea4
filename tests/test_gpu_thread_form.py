"""The one-thread form of the evaluation kernels, beyond the batches that take a
group of lanes per atom (36,864 slots), and at any size by variants 8 and 4: a
configuration keeps its bits whether it is evaluated alone, by groups, or inside
a batch that takes a thread per atom; and a fresh handle's first call, whose
lists are too short and built again, equals its second."""
import numpy as np
import pytest

from paper_2607_06969_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MODELS = {"gst": W.hp_gst, "table2": W.hp_table2}
GROUP_SLOTS = 36864  # nep_kernels.hpp: kWaveSlots


def _cluster(n, a, cell):
    s = W.simple_cubic(n=n, spacing=a, sigma=0.05, seed=5, species_count=3)
    s.cells = np.eye(3)[None] * cell
    s.pos = (s.pos + 0.25 * cell).astype(np.float32).astype(np.float64)
    return s


@pytest.mark.parametrize("model", sorted(MODELS))
def test_alone_equals_inside_a_thread_form_batch(model):
    from paper_2607_06969_amd import nep
    hp = MODELS[model]()
    m = nep.NepModel(hp, W.random_params(hp, 12))
    s = W.concat_systems([W.rocksalt_gst(8, seed=21), W.rocksalt_gst(36, seed=22), W.rocksalt_gst(14, seed=23)])
    assert s.n_atoms > GROUP_SLOTS
    b = nep.Batch.from_system(s)
    full, q = m.compute(b, atom_energy=True, atom_virial=True), m.descriptors(b)
    for c in (0, 2):
        assert s.config(c).n_atoms + 192 < GROUP_SLOTS
        bc = nep.Batch.from_system(s.config(c))
        one = m.compute(bc, atom_energy=True, atom_virial=True)
        a, e = int(s.atom_off[c]), int(s.atom_off[c + 1])
        for k in ("F", "Ei", "Wi"):
            assert torch.equal(one[k], full[k][a:e]), k
        assert torch.equal(one["E"], full["E"][c:c + 1]) and torch.equal(one["V"], full["V"][c:c + 1])
        assert torch.equal(m.descriptors(bc), q[a:e])


# 34^3 = 39,304 atoms take a thread each, 7^3 with the variants that do at any size
@pytest.mark.parametrize("n,a,cell,variants", [(34, 1.9, 700.0, (0, 0)), (7, 1.7, 90.0, (8, 4)), (7, 1.7, 90.0, (7, 5))])
@pytest.mark.parametrize("what", ["compute", "descriptors", "loss_grad", "backward_params"])
def test_first_call_on_too_small_lists(n, a, cell, variants, what):
    from paper_2607_06969_amd import nep
    hp = W.hp_table2()
    m = nep.NepModel(hp, W.random_params(hp, 3))
    m.set_variants(*variants)
    b = nep.Batch.from_system(_cluster(n, a, cell))
    assert variants != (0, 0) or b.n_atoms > GROUP_SLOTS
    print(f"[thread form] {what} {b.n_atoms} atoms", flush=True)
    lab = [torch.linspace(-1, 1, b.n_cfg, dtype=torch.float64, device="cuda"),
           torch.linspace(-1, 1, 3 * b.n_atoms, device="cuda").view(b.n_atoms, 3).contiguous(),
           torch.linspace(-1, 1, 9 * b.n_cfg, dtype=torch.float64, device="cuda").view(-1, 9).contiguous()]
    call = {"compute": lambda: tuple(m.compute(b, atom_energy=True, atom_virial=True).values()),
            "descriptors": lambda: (m.descriptors(b),), "loss_grad": lambda: m.loss_grad(b, *lab),
            "backward_params": lambda: (m.backward_params(b, *lab),)}[what]
    one = [t.clone() for t in call()]
    for x, y in zip(one, call()):
        assert torch.isfinite(x).all() and torch.equal(x, y)
