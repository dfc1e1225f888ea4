"""Float64 calls choose between a wavefront per atom and passes by the batch's
size and by its own lists: molecules (more angular pairs than one chunk, few
others) leave the wavefront form earlier.  A batch beyond such a limit against
its parts within it, energies and forces of the parts side by side and the
gradient their sum.  Both are float64 sums of the same terms in another order:
1e-10 relative."""
import numpy as np
import pytest

from paper_2607_06969_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _molecules(n_cfg, seed):
    """n_cfg open cells of 20 atoms, 3 x 3 x 3 sites 2.3 A apart less seven."""
    rng = np.random.default_rng(seed)
    g = np.stack(np.meshgrid(*[np.arange(3)] * 3, indexing="ij"), axis=-1).reshape(-1, 3) * 2.3 + 15.0
    pos = np.stack([g[rng.permutation(27)[:20]] for _ in range(n_cfg)]) + rng.normal(0.0, 0.1, (n_cfg, 20, 3))
    pos = pos.reshape(-1, 3).astype(np.float32).astype(np.float64)
    return W.System(pos, rng.integers(0, 3, len(pos)).astype(np.int32), np.repeat(np.eye(3)[None] * 35.0, n_cfg, 0),
                    np.arange(n_cfg + 1, dtype=np.int64) * 20, {}, np.zeros((n_cfg, 3), dtype=np.int32))


def _part(s, lo, hi):
    return W.System(s.pos[20 * lo:20 * hi], s.species[20 * lo:20 * hi], s.cells[lo:hi], s.atom_off[:hi - lo + 1], {},
                    s.pbc[lo:hi])


def _rel(a, b):
    return float((a - b).norm() / b.norm())


# 22,000 atoms: gradient in passes; 34,000: evaluation too; 50,000: whatever the lists are
@pytest.mark.parametrize("n_cfg", [1100, 1700, 2500])
def test_molecules(n_cfg):
    from paper_2607_06969_amd import nep
    hp = W.hp_table2()
    m = nep.NepModel(hp, W.random_params(hp, 5))
    P = torch.as_tensor(W.random_params(hp, 5), dtype=torch.float64, device="cuda")
    s, n = _molecules(n_cfg, 1), 2 if n_cfg < 2000 else 4
    b = nep.Batch.from_system(s)
    bs = [nep.Batch.from_system(_part(s, n_cfg * k // n, n_cfg * (k + 1) // n)) for k in range(n)]
    longest = [int(m.neighbors(b, w, cap=1)[0].max()) for w in (0, 1)]
    assert longest[0] < 32 and longest[1] > 16
    rng = np.random.default_rng(6)
    seeds = [[torch.as_tensor(rng.normal(size=k), device="cuda") for k in ((x.n_cfg,), (x.n_atoms, 3), (x.n_cfg, 9))]
             for x in bs]
    print(f"[float64 rule] {b.n_atoms} atoms", flush=True)
    whole = m.compute64(b, P, atom_energy=True)
    parts = [m.compute64(x, P, atom_energy=True) for x in bs]
    for k in ("E", "F", "V", "Ei"):
        assert _rel(whole[k], torch.cat([p[k] for p in parts])) <= 1e-10, k
    g = m.backward_params64(b, P, *[torch.cat(t) for t in zip(*seeds)])
    gs = sum(m.backward_params64(x, P, *s) for x, s in zip(bs, seeds))
    assert torch.isfinite(g).all() and _rel(g, gs) <= 1e-10
