"""The parameter gradient of small batches is one kernel, a wavefront per atom;
larger batches run it in passes.  Where that kernel changes its path (lists of
several rounds, more angular pairs than it holds at a time, no pairs at all, a
species without atoms, a single atom) it is compared with the FP64 oracle, and
both sides of the size rule with each other: a gradient is the sum of its
configurations' gradients, so a batch above the limit equals the sum of its
halves below it.

Tolerances: those of the existing comparisons with the oracle, 1e-4 relative RMS
in float32 and 1e-9 in float64; sums of two results twice that."""
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


def _absent(t):
    s = _lattice(6, 2.9, 6, t)
    s.species[:] = t - 1
    return s


MODELS = {"small": W.hp_small_single, "gst": W.hp_gst, "table2": W.hp_table2}
SYSTEMS = {
    # about 185 (293) radial and 54 (106) angular neighbours
    "dense": lambda t: _lattice(9, 1.7, 1, t),
    "slab_and_alone": lambda t: W.concat_systems([_lattice(6, 2.9, 3, t, [1, 1, 0]), _alone(t), _lattice(6, 3.1, 4, t)]),
    "one_species_only": _absent,
    "alone": _alone,
}


def _rel(a, b):
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)


def _seeds(s, seed):
    rng = np.random.default_rng(seed)
    return (rng.normal(size=s.n_cfg), (1e-3 * rng.normal(size=(s.n_atoms, 3))).astype(np.float32).astype(np.float64),
            1e-3 * rng.normal(size=(s.n_cfg, 9)))


def _gradients(m, p, s, seeds):
    from paper_2607_06969_amd import nep
    b = nep.Batch.from_system(s)
    eb, lam, mu = (torch.tensor(x, device="cuda") for x in seeds)
    P = torch.tensor(p, dtype=torch.float64, device="cuda")
    return (m.backward_params(b, eb, lam.float().contiguous(), mu).cpu().numpy().astype(np.float64),
            m.backward_params64(b, P, eb, lam, mu).cpu().numpy())


@pytest.mark.parametrize("model", sorted(MODELS))
@pytest.mark.parametrize("system", sorted(SYSTEMS))
def test_gradient_matches_oracle(oracle_lib, model, system):
    from paper_2607_06969_amd import nep
    hp = MODELS[model]()
    s = SYSTEMS[system](hp.n_species)
    p = W.random_params(hp, 11)
    seeds = _seeds(s, 3)
    # labels that make the oracle's loss have these seeds (pooled form)
    ref = oracle_lib.evaluate(hp, p, s, nbr_mode=2)
    n = np.diff(s.atom_off).astype(np.float64)
    w = (1.0, 1.0, 0.1)
    Er = ref["E"] - seeds[0] * s.n_cfg * n ** 2 / 2.0
    Fr = ref["F"] - seeds[1] * 3.0 * s.n_atoms / 2.0
    Vr = ref["V"].reshape(-1, 9) - seeds[2] * 9.0 * s.n_cfg * n[:, None] ** 2 / (2.0 * w[2])
    _, g = oracle_lib.loss_grad(hp, p, s, Er, Fr, Vr, weights=w, loss_form=0, nbr_mode=2)
    print(f"[train wave] {model} {system}: N={s.n_atoms}", flush=True)
    g32, g64 = _gradients(nep.NepModel(hp, p), p, s, seeds)
    assert _rel(g32, g) <= 1e-4, _rel(g32, g)
    assert _rel(g64, g) <= 1e-9, _rel(g64, g)


def test_both_sides_of_the_size_rule():
    from paper_2607_06969_amd import nep
    hp = W.hp_gst()
    p = W.random_params(hp, 12)
    m = nep.NepModel(hp, p)
    halves = [_lattice(n, 3.0, 20 + n, 3) for n in (28, 30)]  # 21,952 + 27,000 atoms
    seeds = [_seeds(s, n) for n, s in enumerate(halves)]
    both = W.concat_systems(halves + halves[:1])               # 70,904 atoms
    print(f"[train wave] N={both.n_atoms}", flush=True)
    g32, g64 = _gradients(m, p, both, [np.concatenate(x) for x in zip(*(seeds + seeds[:1]))])
    parts = [_gradients(m, p, s, x) for s, x in zip(halves, seeds)]
    for got, one, two, tol in ((g32, parts[0][0], parts[1][0], 2e-4), (g64, parts[0][1], parts[1][1], 2e-9)):
        assert _rel(got, 2 * one + two) <= tol, _rel(got, 2 * one + two)
