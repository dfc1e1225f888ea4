"""A run of MD replays graphs of eight steps and, for what is left, of one: runs of
any length equal the same steps taken one at a time, bit for bit, across list
rebuilds (small skin) and the checkpoint after 32 steps."""
import numpy as np
import pytest

from paper_2607_06969_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _md():
    from paper_2607_06969_amd import nep
    hp = W.hp_gst()
    s = W.concat_systems([W.rocksalt_gst(8, seed=31), W.rocksalt_gst(10, seed=32)])
    m = nep.NepModel(hp, W.random_params(hp, 3, std=0.05))
    m.set_variants(0, 0)
    v = W.maxwell_boltzmann(s.species, W.MASSES_GST, 600.0, seed=5)
    b = nep.Batch.from_system(s)
    return nep.NepMD(m, b, torch.as_tensor(v, dtype=torch.float32, device="cuda"), W.MASSES_GST, dt_fs=2.0, skin=0.3)


@pytest.mark.parametrize("steps", [1, 7, 8, 9, 32, 43])
def test_any_length_equals_single_steps(steps):
    one, run = _md(), _md()
    for _ in range(steps):
        one.step(1)
    run.step(steps)
    a, b = one.state(), run.state()
    for k in ("pos", "vel", "F", "Epot", "Ekin", "V"):
        assert torch.equal(a[k], b[k]), k
    assert one.stats() == run.stats()
