"""A dense cluster in a large empty cell: the first call's list capacities come
from the mean density and are far too small, so the evaluation launched on the
truncated lists has to be repeated on the regrown ones.  The first call on a
fresh handle must equal the second bit for bit, in both forms of the kernels
and for every entry point that launches work before the lists are checked."""
import numpy as np
import pytest

from paper_2607_06969_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _cluster(n, a, cell):
    s = W.simple_cubic(n=n, spacing=a, sigma=0.05, seed=5, species_count=3)
    s.cells = np.eye(3)[None] * cell
    s.pos = (s.pos + 0.25 * cell).astype(np.float32).astype(np.float64)
    return s


def _calls(m, b):
    n = b.n_atoms
    lab = [torch.linspace(-1, 1, b.n_cfg, dtype=torch.float64, device="cuda"),
           torch.linspace(-1, 1, 3 * n, device="cuda").view(n, 3).contiguous(),
           torch.linspace(-1, 1, 9 * b.n_cfg, dtype=torch.float64, device="cuda").view(-1, 9).contiguous()]
    yield "compute", lambda: tuple(m.compute(b, atom_energy=True, atom_virial=True).values())
    yield "descriptors", lambda: (m.descriptors(b),)
    yield "loss_grad", lambda: m.loss_grad(b, *lab)
    yield "backward_params", lambda: (m.backward_params(b, lab[0], lab[1], lab[2]),)


@pytest.mark.parametrize("n,a,cell", [(7, 1.7, 90.0), (30, 1.9, 600.0)])
@pytest.mark.parametrize("what", ["compute", "descriptors", "loss_grad", "backward_params"])
def test_first_call_on_too_small_lists(n, a, cell, what):
    from paper_2607_06969_amd import nep
    hp = W.hp_table2()
    m = nep.NepModel(hp, W.random_params(hp, 3))
    b = nep.Batch.from_system(_cluster(n, a, cell))
    print(f"[first call] {what} {b.n_atoms} atoms", flush=True)
    call = dict(_calls(m, b))[what]
    one = [t.clone() for t in call()]
    two = call()
    for x, y in zip(one, two):
        assert torch.isfinite(x).all() and torch.equal(x, y)
