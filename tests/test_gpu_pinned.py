"""The library's pinned host memory (tables on their way to the GPU, list flags
on their way back) is taken when a handle is created and kept until the process
ends: no later call maps or unmaps host memory, the allocation-free entry point
does not from its first call on, and handles that come and go reuse it.  Tables
too large for a handle's block take another way to the GPU with the same
results, and calls of several models may alternate on the allocation-free
workspace."""
import numpy as np
import pytest

from paper_2607_06969_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _host_maps():
    """Address ranges that the GPU driver has mapped into this process (pinned host memory is among them)."""
    with open("/proc/self/maps") as f:
        return {ln.split()[0] for ln in f if "/dev/dri" in ln or "/dev/kfd" in ln}


def _clusters(n_cfg, n, seed):
    """n_cfg clusters of n atoms, each in a 16 A cell of its own without periodic directions."""
    rng = np.random.default_rng(seed)
    g = np.stack(np.meshgrid(*[np.arange(2)] * 3, indexing="ij"), axis=-1).reshape(-1, 3)[:n] * 2.8 + 6.0
    pos = (g[None] + rng.normal(0.0, 0.1, (n_cfg, n, 3))).reshape(-1, 3).astype(np.float32).astype(np.float64)
    return W.System(pos, rng.integers(0, 3, n_cfg * n).astype(np.int32), np.repeat(np.eye(3)[None] * 16.0, n_cfg, 0),
                    np.arange(n_cfg + 1, dtype=np.int64) * n, {}, np.zeros((n_cfg, 3), dtype=np.int32))


def _batch(s):
    from paper_2607_06969_amd import nep
    return nep.Batch.from_system(s)


def _model(seed=7):
    from paper_2607_06969_amd import nep
    hp = W.hp_gst()
    return nep.NepModel(hp, W.random_params(hp, seed))


def test_noalloc_maps_no_host_memory():
    few, more, many = (_batch(_clusters(n, 4, 2)) for n in (2, 90, 400))
    # code objects, the static workspace and torch's own memory are in place after this
    warm = _model()
    for b in (few, more, many):
        warm.compute(b)
    warm.compute(few, noalloc=True)
    torch.cuda.synchronize()
    m = _model()
    before = _host_maps()
    for b in (few, more, many, few):
        m.compute(b, noalloc=True)
        torch.cuda.synchronize()
        assert _host_maps() == before


@pytest.mark.parametrize("n_cfg", [1, 300, 1500])
@pytest.mark.parametrize("noalloc", [True, False])
def test_tables_of_any_size(n_cfg, noalloc):
    """1,500 configurations have some 370 KB of tables, more than a handle's block."""
    m = _model()
    s = _clusters(n_cfg, 4, 3)
    out = m.compute(_batch(s), noalloc=noalloc)
    for c in sorted({0, n_cfg // 2, n_cfg - 1}):
        one = m.compute(_batch(s.config(c)))
        assert torch.equal(out["E"][c:c + 1], one["E"]) and torch.equal(out["V"][c:c + 1], one["V"])
        assert torch.equal(out["F"][4 * c:4 * c + 4], one["F"])


def test_models_alternate_on_the_static_workspace():
    a, b = _model(7), _model(8)
    x, y = _batch(W.rocksalt_gst(8, seed=31)), _batch(_clusters(40, 6, 4))
    want = {(i, j): [t.clone() for t in m.compute(q).values()] for i, m in enumerate((a, b)) for j, q in enumerate((x, y))}
    for i, j in [(0, 0), (1, 1), (0, 1), (1, 0), (1, 1), (0, 0), (0, 0), (1, 0)]:
        m, q = (a, b)[i], (x, y)[j]
        got = m.compute(q, noalloc=True)
        own = m.compute(q)
        for t, u, v in zip(want[i, j], got.values(), own.values()):
            assert torch.equal(t, u) and torch.equal(t, v)


def test_handles_that_come_and_go():
    s = W.rocksalt_gst(8, seed=32)
    b, ref, held = _batch(s), None, None
    for k in range(40):
        m = _model()
        out = [t.clone() for t in m.compute(b).values()]
        ref = ref or out
        assert all(torch.equal(t, u) for t, u in zip(ref, out))
        del m
