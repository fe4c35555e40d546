"""qcx_set_memory_limit is host bookkeeping: it may be called while the
context's stream is being captured, also by a context that holds buffers of the
panel route, and those are freed once something needs their room."""
import numpy as np
import pytest

from synth import make_si_ng113
from tests.gpu_helpers import set_inputs

pytestmark = pytest.mark.gpu


def test_limit_while_capturing():
    import torch

    from paper_2603_12326_amd import Context

    wl = make_si_ng113(n_q=1, n_w=300, kgrid=5)
    s = torch.cuda.Stream()
    c = Context(0, stream=s.cuda_stream)
    set_inputs(c, wl)
    c.pair_density(wl.G_int)
    c.chi0(wl.w_eV, wl.eta_eV, "split_bf16")
    assert c.bulk_config()["stages"] == 0
    c.eps_inv(True)
    want = c.loss()
    x = torch.zeros(1000, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    used = c.memory_used()
    with torch.cuda.graph(g, stream=s):
        x += 1
        c.set_memory_limit(used + (64 << 20))
        x += 1
    for _ in range(3):
        g.replay()
    torch.cuda.synchronize()
    assert bool((x == 6).all())
    # more than the 64 MiB are needed (without the partials of tuning), and found
    c.set_autotune(0)
    w = np.linspace(0.0, 40.0, 500)
    c.chi0(w, wl.eta_eV, "split_bf16")
    assert c.bulk_config()["stages"] != 0
    c.eps_inv(True)
    assert np.all(np.isfinite(c.loss()))
    assert c.memory_used() <= used + (64 << 20)
    c.set_memory_limit(0)
    c.chi0(wl.w_eV, wl.eta_eV, "split_bf16")
    c.eps_inv(True)
    assert np.array_equal(c.loss(), want)
    c.close()
