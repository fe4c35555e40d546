"""The panel route where its work comes in pieces: several ranges of pairs,
coefficients in several chunks of frequencies, transition counts off every
multiple of the kernels' steps.  Every case has to take panels; the reference is
the direct sum in FP64 (the same call under a memory cap too large to bind)."""
import numpy as np
import pytest

from synth import make_si_ng113
from synth.generator import _sorted_g

pytestmark = pytest.mark.gpu

# of the largest |chi0|, as for a single piece: FP64 sums of about 1e4 terms
# through 32-term series; FP32 sums of at most 1024 steps of 24-bit operands
_BAR = dict(fp64=1e-12, fp32=2e-6, split_bf16=2e-6)


@pytest.fixture(scope="module")
def case():
    wl = make_si_ng113(n_q=1, n_w=400, kgrid=6)
    r = np.arange(-6, 7)
    G = _sorted_g(np.stack(np.meshgrid(r, r, r, indexing="ij"), axis=-1).reshape(-1, 3), wl.cell.lat)
    return wl, G


def _chi(case, n_g, w, eta, precision, direct, k=slice(None), bands=None):
    import torch

    from paper_2603_12326_amd import Context

    wl, G = case
    st, b = wl.states(0), wl.basis
    n_occ, cols = (wl.n_occ, slice(None)) if bands is None else bands
    c = Context(0)
    if direct:
        c.set_memory_limit(1 << 40)
    c.set_cell_basis(wl.cell.lat, wl.cell.xyz, b.shell_atom, b.shell_l, b.shell_exp, 1, 1)
    c.set_states(st.q_cart, wl.k_frac[k], n_occ, st.C_k[k][:, :, cols], st.E_k[k][:, cols], st.C_kq[k][:, :, cols],
                 st.E_kq[k][:, cols])
    c.pair_density(G[:n_g])
    chi = torch.empty((len(w), n_g, n_g), dtype=torch.complex128, device="cuda")
    c.chi0(w, eta, precision, True, chi)
    c.sync()
    panels = c.bulk_config()["stages"] == 0
    c.close()
    return chi, panels


def _check(case, n_g, w, eta, precision, **kw):
    import torch

    got, panels = _chi(case, n_g, w, eta, precision, False, **kw)
    ref, _ = _chi(case, n_g, w, eta, "fp64", True, **kw)
    assert panels
    if precision == "fp64":
        assert not torch.equal(got, ref)  # panels, not the same sum
    err = float((got - ref).abs().max() / ref.abs().max())
    print(f"{precision} {n_g} G {len(w)} w: {err:.2e}")
    assert err <= _BAR[precision]


@pytest.mark.parametrize("precision,n_g,n_w", [("fp64", 181, 230), ("fp64", 259, 90), ("split_bf16", 301, 97),
                                               ("fp32", 301, 64)])
def test_several_ranges_of_pairs(case, precision, n_g, n_w):
    """FP64 moments hold about 8,400 pairs at a time here, the others 22,000."""
    _check(case, n_g, np.linspace(0.0, 60.0, n_w), 0.1, precision)


def test_ranges_and_chunks_of_frequencies(case):
    """About 1,000 panels a side: the pairs in 2 ranges and the coefficients in 2
    chunks of frequencies."""
    _check(case, 161, np.linspace(0.0, 300.0, 6000), 0.3, "split_bf16")


def test_fp32_splits_that_do_not_fit(case):
    """18 splits of 2.5 GB: the FP32 mode sums directly."""
    _, panels = _chi(case, 161, np.linspace(0.0, 300.0, 6000), 0.3, "fp32", False)
    assert not panels


@pytest.mark.parametrize("precision,n_g,n_w,eta", [("fp64", 65, 400, 0.1), ("fp32", 65, 400, 0.1),
                                                   ("split_bf16", 113, 330, 0.1), ("fp64", 30, 211, 0.2)])
@pytest.mark.parametrize("n_k", [211, 205])
def test_odd_transition_counts(case, precision, n_g, n_w, eta, n_k):
    """3 occupied and 15 empty bands at an odd number of k points: 90 n_k
    transitions, sides of 45 n_k (odd)."""
    _check(case, n_g, np.linspace(0.0, 50.0, n_w), eta, precision, k=slice(0, n_k), bands=(3, slice(1, 19)))


def test_few_transitions(case):
    """1,386 transitions and a wide broadening: panels of a few transitions each."""
    _check(case, 181, np.linspace(0.0, 60.0, 4000), 3.0, "split_bf16", k=slice(0, 33), bands=(3, slice(1, 11)))
