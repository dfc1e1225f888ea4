"""Gradients of batches near the limits of the one-pass kernel with a rare
species: its few slots get one block, so each wavefront sums more atoms than
those of the others (16 in float32, 80 in float64) before the float64 sum.
Float32 against float64 at the same parameters, for the whole gradient and for
the rare species' own entries: 1e-4 relative, the bar of the comparisons with
the oracle."""
import numpy as np
import pytest

from paper_2607_06969_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# 19,756 atoms: one pass in float32 and float64; 41,990: passes in float32, one pass in float64
@pytest.mark.parametrize("n,rare", [(28, 1), (28, 40), (36, 300)])
def test_rare_species(n, rare):
    from paper_2607_06969_amd import nep
    hp = W.hp_gst()
    s = W.rocksalt_gst(n, seed=61)
    s.species[:] = W.TE
    s.species[np.random.default_rng(62).permutation(s.n_atoms)[:rare]] = W.SB
    p = W.random_params(hp, 63)
    m = nep.NepModel(hp, p)
    b = nep.Batch.from_system(s)
    rng = np.random.default_rng(64)
    eb, lam, mu = rng.normal(size=1), 1e-3 * rng.normal(size=(s.n_atoms, 3)), 1e-3 * rng.normal(size=(1, 9))
    lam = lam.astype(np.float32).astype(np.float64)
    eb, lam, mu = (torch.tensor(x, device="cuda") for x in (eb, lam, mu))
    print(f"[rare species] {s.n_atoms} atoms, {rare} of a kind", flush=True)
    g32 = m.backward_params(b, eb, lam.float().contiguous(), mu).double()
    g64 = m.backward_params64(b, torch.tensor(p, dtype=torch.float64, device="cuda"), eb, lam, mu)
    mlp = hp.n_hidden * hp.dim + 2 * hp.n_hidden + 1
    own = slice(hp.n_params() - (3 - W.SB) * mlp, hp.n_params() - (2 - W.SB) * mlp)
    absent = slice(hp.n_params() - 3 * mlp, hp.n_params() - 2 * mlp)
    for part in (slice(None), own):
        assert float(g64[part].norm()) > 0
        assert float((g32[part] - g64[part]).norm() / g64[part].norm()) <= 1e-4
    assert not g32[absent].any() and not g64[absent].any()
