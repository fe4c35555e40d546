"""The energy panels' buffers, which a context keeps for its next call, make
room when the device runs out of memory for something else: calls that fitted
without them still do."""
import numpy as np
import pytest

from synth import make_si_ng113
from tests.gpu_helpers import set_inputs

pytestmark = pytest.mark.gpu

W = np.linspace(0.0, 60.0, 20000)  # eps of 113 G: 4.1 GB
N_G = 113


@pytest.fixture(scope="module")
def wl():
    return make_si_ng113(n_q=1, n_w=400, kgrid=6)


def _free():
    import torch

    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def _chi0(wl):
    """A context whose chi0 ran through panels, and the size of its buffers."""
    from paper_2603_12326_amd import Context

    c = Context(0)
    set_inputs(c, wl)
    c.pair_density(wl.G_int[:N_G])
    before = c.memory_used()
    c.chi0(W, wl.eta_eV, "split_bf16")
    c.sync()
    assert c.bulk_config()["stages"] == 0
    return c, before


def _leave(n):
    """Fill the device but for n bytes."""
    import torch

    assert n > 1 << 30
    f = _free()
    return torch.empty(f - n, dtype=torch.uint8, device="cuda")


def test_inversion_after_panels(wl):
    import torch

    c, _ = _chi0(wl)
    c.eps_inv(True)
    want = c.loss()
    c.close()
    c, before = _chi0(wl)
    used = c.memory_used()
    eps = 16 * len(W) * N_G * N_G
    print(f"chi0 {(used - before) / 1e9:.2f} GB, eps {eps / 1e9:.2f} GB")
    assert used - before > 4 * eps // 2
    fill = _leave(eps - (1 << 30))
    c.eps_inv(True)
    got = c.loss()
    assert c.memory_used() < used + eps
    del fill
    torch.cuda.empty_cache()
    assert np.array_equal(got, want)
    # and the next call takes panels again
    c.chi0(W, wl.eta_eV, "split_bf16")
    assert c.bulk_config()["stages"] == 0
    c.eps_inv(True)
    assert np.array_equal(c.loss(), want)
    c.close()


def test_batch_after_panels(wl):
    import torch

    from paper_2603_12326_amd import Context, qcx

    w = W[::5]
    out = torch.empty((len(w), N_G), dtype=torch.float64, device="cuda")
    items = [dict(ctx=0, w_eV=w, eta_eV=wl.eta_eV, loss_out=out)]

    def context():
        c = Context(0)
        c.set_autotune(0)
        set_inputs(c, wl)
        c.pair_density(wl.G_int[:N_G])
        return c

    c = context()
    f = _free()
    qcx.run_batch([c], items)
    qcx.batch_sync(c)
    need = f - _free()
    want = out.clone()
    c.close()
    c, _ = _chi0(wl)
    c.set_autotune(0)
    print(f"batch {need / 1e9:.2f} GB")
    fill = _leave(need - (1 << 29))
    out.zero_()
    qcx.run_batch([c], items)
    qcx.batch_sync(c)
    del fill
    torch.cuda.empty_cache()
    assert torch.equal(out, want)
    c.close()


def test_panels_leave_half_of_what_is_free(wl):
    """With little memory left the transitions are summed directly."""
    import torch

    from paper_2603_12326_amd import Context

    c = Context(0)
    set_inputs(c, wl)
    c.pair_density(wl.G_int[:N_G])
    c.set_autotune(0)
    fill = _leave(3 << 30)
    c.chi0(W[::20], wl.eta_eV, "split_bf16")  # panels of more than 1.5 GiB
    assert c.bulk_config()["stages"] != 0
    c.sync()
    del fill
    torch.cuda.empty_cache()
    c.chi0(W[::20], wl.eta_eV, "split_bf16")
    assert c.bulk_config()["stages"] == 0
    c.sync()
    c.close()
