"""qcx_mlp_infer with the networks on one stream and the contexts on others:
calls that follow each other without a wait, each with rows of its own to
place."""
import numpy as np
import pytest

from synth import make_si_ng113
from synth.surrogate import mlp_init

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ctx", [1, 2])
def test_calls_in_a_row(n_ctx):
    """Three calls with different tolerances (other rejected frequencies, other
    frequency counts), waited for one by one and then not until the end: the
    same bits.  Device states, so that nothing in between waits; the method's
    rows take longer than the networks of the next call.  Two contexts take
    turns on streams of their own."""
    import torch

    from paper_2603_12326_amd import Context, Mlp

    wl = make_si_ng113(n_q=1, n_w=8, kgrid=4)
    st, b = wl.states(0), wl.basis
    dev = [torch.as_tensor(x, device="cuda") for x in (wl.k_frac, st.C_k, st.E_k, st.C_kq, st.E_kq)]
    streams = [torch.cuda.Stream() for _ in range(1 + n_ctx)]
    torch.cuda.synchronize()
    net = Context(0, stream=streams[0].cuda_stream)
    m = Mlp(net, 3)
    for k in range(3):
        m.set_params(k, mlp_init(80 + k))
    m.set_encoding(6.0, 60.0, np.asarray(wl.cell.lat, np.float64), -3.0, 2.0, 1.0)
    ctxs = [Context(0, stream=s.cuda_stream) for s in streams[1:]]
    for c in ctxs:
        c.set_cell_basis(wl.cell.lat, wl.cell.xyz, b.shell_atom, b.shell_l, b.shell_exp, 1, 1)
        c.set_states(st.q_cart, dev[0], wl.n_occ, *dev[1:])
        c.sync()
    G = np.asarray(wl.G_int, np.int32)
    lists = [np.linspace(0.2, 59.0, n) for n in (240, 180, 260)]
    # tolerances at which about 80%, 30% and 60% of the rows are recomputed
    tols = []
    for w, keep in zip(lists, (0.2, 0.7, 0.4)):
        e = torch.empty((len(w), len(G)), dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        assert m.infer(ctxs[0], G, w, wl.eta_eV, 1e300, "fp64", err_out=e)[2] == 0
        torch.cuda.synchronize()
        tols.append(float(np.quantile(e.cpu().numpy().max(axis=1), keep)))

    def calls(wait):
        out = [torch.full((len(w), len(G)), -7.0, dtype=torch.float64, device="cuda") for w in lists]
        torch.cuda.synchronize()
        n = []
        for i, (w, tol) in enumerate(zip(lists, tols)):
            n.append(m.infer(ctxs[i % n_ctx], G, w, wl.eta_eV, tol, "fp64", loss_out=out[i])[2])
            if wait:
                torch.cuda.synchronize()
        for c in [net] + ctxs:
            c.sync()
        torch.cuda.synchronize()
        return n, [o.cpu().numpy() for o in out]

    calls(True)
    n0, want = calls(True)
    assert len(set(n0)) == 3 and min(n0) > 0
    for _ in range(3):
        n1, got = calls(False)
        assert n1 == n0
        for a, w in zip(got, want):
            assert np.array_equal(a, w)
    m.close()
    for c in ctxs + [net]:
        c.close()
