"""A call that refuses its input (a non-finite position, a species out of range)
leaves every output array as it was, and nothing that it has launched is still
running when it returns: the evaluation is launched before the list flags that
tell of such an input are known.  Batches for the lane-group and the one-thread
form of the kernels, descriptor variants with the network in the kernel and
apart, and each entry point that launches work ahead of the flags."""
import ctypes as C

import numpy as np
import pytest

from paper_2607_06969_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MARK = 12345.5


def _calls(m, b, outs):
    from paper_2607_06969_amd._lib import _host_f64, _ptr, _stream, load
    keep, off, cells, pbc = b._meta()
    n, nc = b.n_atoms, b.n_cfg

    def new(k, dtype):
        outs.append(torch.full((k,), MARK, dtype=dtype, device="cuda"))
        return _ptr(outs[-1])

    f, d = torch.float32, torch.float64
    head = (m._h, nc, off, cells, pbc, _ptr(b.pos), _ptr(b.species))
    refs = [torch.zeros(nc, dtype=d, device="cuda"), torch.zeros(3 * n, device="cuda"),
            torch.zeros(9 * nc, dtype=d, device="cuda")]
    w, pw = _host_f64((1.0, 1.0, 0.1))
    L, st, held = load(), _stream(), (keep, w, refs)
    return held, {
        "compute": lambda: L.nepmi_compute(*head, new(nc, d), new(3 * n, f), new(9 * nc, d), new(n, f), new(9 * n, f), st),
        "noalloc": lambda: L.nepmi_compute_noalloc(*head, new(nc, d), new(3 * n, f), new(9 * nc, d), new(n, f),
                                                   new(9 * n, f), st),
        "descriptors": lambda: L.nepmi_descriptors(*head, new(n * m.dim, f), st),
        "backward_params": lambda: L.nepmi_backward_params(*head, *map(_ptr, refs), new(m.n_params, f), st),
        "loss_grad": lambda: L.nepmi_loss_grad(*head, *map(_ptr, refs), pw, 0, new(4, d), new(m.n_params, f), st),
    }


def _batch(size, fault):
    from paper_2607_06969_amd import nep
    parts = {"small": [W.rocksalt_gst(6, seed=51), W.rocksalt_gst(8, seed=52)],
             "large": [W.rocksalt_gst(8, seed=53), W.rocksalt_gst(36, seed=54)]}[size]
    b = nep.Batch.from_system(W.concat_systems(parts))
    if fault == "nan":
        b.pos[b.n_atoms // 2, 1] = float("nan")
    elif fault == "species":
        b.species[b.n_atoms // 3] = 3
    return b


CALLS = ["compute", "descriptors", "backward_params", "loss_grad"]
FORMS = [("small", (0, 0)), ("small", (5, 4)), ("large", (0, 0)), ("large", (7, 0))]


# (the large batch is beyond the workspace of the allocation-free call)
@pytest.mark.parametrize("what,size,variants", [(w, *f) for w in CALLS for f in FORMS] +
                         [("noalloc", *f) for f in FORMS[:2]])
def test_refused_call_writes_nothing(what, size, variants):
    from paper_2607_06969_amd import nep
    from paper_2607_06969_amd._lib import INVALID_ARG, NAN_DETECTED
    hp = W.hp_gst()
    m = nep.NepModel(hp, W.random_params(hp, 13))
    m.set_variants(*variants)
    for fault, code in (("nan", NAN_DETECTED), ("species", INVALID_ARG)):
        b, outs = _batch(size, fault), []
        held, calls = _calls(m, b, outs)
        torch.cuda.synchronize()
        rc = calls[what]()
        done = torch.cuda.current_stream().query()
        torch.cuda.synchronize()
        assert rc == code and done
        for t in outs:
            assert bool((t == MARK).all()), f"{fault}: {int((t != MARK).sum())} of {t.numel()} values written"
    # and the same handle works on a good batch
    b, outs = _batch(size, None), []
    held, calls = _calls(m, b, outs)
    assert calls[what]() == 0
    assert all(bool(torch.isfinite(t).all()) and not bool((t == MARK).any()) for t in outs)
