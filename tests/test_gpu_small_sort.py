"""Small batches: one block sorts the atoms and takes the upload of the
configuration tables along if they are small (about 70 configurations); the first
kernel on the lists delivers their flags.  A batch of many tiny configurations
equals its configurations evaluated one by one, bit for bit, on both sides of
that size, in every call that builds lists, and a batch with an invalid species
is refused by each of them without harm to the next call."""
import numpy as np
import pytest

from paper_2607_06969_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _tiny(n_cfg):
    rng = np.random.default_rng(9)
    grid = np.stack(np.meshgrid(*[np.arange(3)] * 3, indexing="ij"), -1).reshape(-1, 3)[:20]
    pos = np.concatenate([2.8 * grid + 4.0 + rng.uniform(-0.3, 0.3, size=(20, 3)) for _ in range(n_cfg)])
    return W.System(pos.astype(np.float32).astype(np.float64), np.zeros(20 * n_cfg, dtype=np.int32),
                    np.repeat(np.eye(3)[None] * 20.0, n_cfg, axis=0), 20 * np.arange(n_cfg + 1, dtype=np.int64))


def _calls(m, b, k):
    """The calls on b, whose configurations carry the seeds of configuration k on."""
    c, n = b.n_cfg, b.n_atoms
    t = lambda *shape: torch.ones(*shape, dtype=torch.float64, device="cuda")
    out = m.compute(b)
    out["q"] = m.descriptors(b)
    out["grad"] = m.backward_params(b, t(c), t(n, 3).float(), t(c, 9))
    out["loss"], _ = m.loss_grad(b, t(c), t(n, 3).float(), t(c, 9))
    return out


@pytest.mark.parametrize("n_cfg", [1, 8, 70, 128, 160])
def test_many_tiny_configurations(n_cfg):
    from paper_2607_06969_amd import nep
    hp = W.hp_small_single()
    m = nep.NepModel(hp, W.random_params(hp, 4))
    s = _tiny(n_cfg)
    out = _calls(m, nep.Batch.from_system(s), 0)
    for c in sorted({0, n_cfg // 2, n_cfg - 1}):
        one = _calls(m, nep.Batch.from_system(s.config(c)), c)
        a = slice(20 * c, 20 * c + 20)
        assert torch.equal(out["E"][c:c + 1], one["E"]) and torch.equal(out["V"][c:c + 1], one["V"])
        assert torch.equal(out["F"][a], one["F"]) and torch.equal(out["q"][a], one["q"])
    assert torch.isfinite(out["grad"]).all() and torch.isfinite(out["loss"]).all()


def test_invalid_species_is_refused_by_every_call():
    from paper_2607_06969_amd import nep
    from paper_2607_06969_amd._lib import NepmiError
    hp = W.hp_small_single()
    m = nep.NepModel(hp, W.random_params(hp, 4))
    good, bad = _tiny(3), _tiny(3)
    bad.species[7] = 5
    want = _calls(m, nep.Batch.from_system(good), 0)
    b = nep.Batch.from_system(bad)
    t = lambda *shape: torch.ones(*shape, dtype=torch.float64, device="cuda")
    for call in (lambda: m.compute(b), lambda: m.descriptors(b),
                 lambda: m.backward_params(b, t(3), t(60, 3).float(), t(3, 9)),
                 lambda: m.loss_grad(b, t(3), t(60, 3).float(), t(3, 9))):
        with pytest.raises(NepmiError):
            call()
        again = _calls(m, nep.Batch.from_system(good), 0)
        for k in want:
            assert torch.equal(again[k], want[k]), k
