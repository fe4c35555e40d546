"""chi0 and the diagonal loss through energy panels against the direct sum over
transitions (the same call under a memory cap too large to bind, which keeps
the direct route), over tile edges, frequency lists and precisions."""
import numpy as np
import pytest

from synth import make_si_ng113
from tests.gpu_helpers import set_inputs

pytestmark = pytest.mark.gpu

# of the largest |chi0|: FP64 sums of ~1e4 terms through 32-term series;
# operands of 22 bits (2^-22 = 2.4e-7 each) and 24-bit sums
_BAR = dict(fp64=1e-12, fp32=2e-6, split_bf16=2e-6)


@pytest.fixture(scope="module")
def wl():
    return make_si_ng113(n_q=1, n_w=400, kgrid=6)


def _chi(wl, G, w, eta, precision, hw64, direct, iq=0):
    import torch

    from paper_2603_12326_amd import Context

    c = Context(0)
    if direct:
        c.set_memory_limit(1 << 40)
    set_inputs(c, wl, iq)
    chi = torch.empty((len(w), len(G), len(G)), dtype=torch.complex128, device="cuda")
    c.pair_density(G)
    c.chi0(w, eta, precision, hw64, chi)
    first = chi.clone()
    c.chi0(w, eta, precision, hw64, chi)  # a second call: tables kept, the same to the bit
    c.sync()
    assert torch.equal(first, chi)
    c.eps_inv(True)
    loss = c.loss()
    loss = loss.cpu().numpy() if hasattr(loss, "cpu") else np.asarray(loss)
    c.close()
    return chi.cpu().numpy(), loss


def _compare(wl, G, w, eta, precision, hw64, panels=None):
    got, loss = _chi(wl, G, w, eta, precision, hw64, False)
    ref, _ = _chi(wl, G, w, eta, "fp64", True, True)
    same, _ = _chi(wl, G, w, eta, precision, hw64, True)
    direct = np.array_equal(got, same)
    assert panels is None or direct != panels  # the route that is meant
    if direct:
        return
    assert np.max(np.abs(got - ref)) <= _BAR[precision] * np.max(np.abs(ref))
    assert np.all(np.isfinite(loss))


@pytest.mark.parametrize("precision", ["split_bf16", "fp32", "fp64"])
@pytest.mark.parametrize("n_g,n_w", [(31, 399), (32, 160), (33, 161), (64, 97), (65, 400), (113, 33), (113, 320)])
def test_tile_edges(wl, n_g, n_w, precision):
    """Pair and row counts on either side of the tiles (8 x 16 G, 128 pairs,
    32 .. 160 rows)."""
    many = n_g * n_w > 64 * 320  # enough work for the panels to be the cheaper route in any precision
    _compare(wl, wl.G_int[:n_g], np.linspace(0.0, 60.0, n_w), 0.1, precision, True, True if many else None)


@pytest.mark.parametrize("precision", ["split_bf16", "fp64"])
@pytest.mark.parametrize("name", ["unsorted", "negative", "repeated", "wide", "shifted"])
def test_frequency_lists(wl, name, precision):
    rng = np.random.default_rng(9)
    w, eta = dict(unsorted=(rng.uniform(0, 50, 200), 0.2), negative=(np.linspace(-20, 30, 200), 0.15),
                  repeated=(np.repeat(np.linspace(0, 40, 60), 4), 0.1), wide=(np.linspace(0, 30, 200), 3.0),
                  shifted=(np.linspace(80, 140, 200), 0.2))[name]
    _compare(wl, wl.G_int[:65], w, eta, precision, True)


@pytest.mark.parametrize("precision", ["split_bf16", "fp32"])
def test_head_and_wings_in_16_bits(wl, precision):
    _compare(wl, wl.G_int[:51], np.linspace(0.0, 60.0, 300), 0.1, precision, False)


@pytest.mark.parametrize("n_g", [40, 113])
def test_one_energy(wl, n_g):
    """Every transition at one energy: one panel holds them all (several
    entries of the bulk's binning), the others none."""
    import copy

    w1 = copy.copy(wl)
    st = wl.states(0)
    E = np.broadcast_to(np.where(np.arange(wl.n_bands) < wl.n_occ, -1.0, 9.0), st.E_k.shape).copy()
    one = copy.copy(st)
    one.E_k, one.E_kq = E, E.copy()
    w1.states = lambda iq: one
    for precision in ("split_bf16", "fp32", "fp64"):
        _compare(w1, wl.G_int[:n_g], np.linspace(0.0, 40.0, 200), 0.1, precision, True)


def test_few_frequencies_stay_direct(wl):
    _compare(wl, wl.G_int[:27], np.array([3.0, 9.0]), 0.1, "split_bf16", True, panels=False)


@pytest.mark.parametrize("n_g", [700, 4133])
def test_diagonal_loss(wl, n_g):
    """The FP64 diagonal, one chunk of 4096 G and a ragged second one.  Loss =
    Im eps / |eps|^2 of chi0 good to 1e-12: bar 1e-10 of each largest loss."""
    from paper_2603_12326_amd import Context
    from synth.generator import _sorted_g

    r = np.arange(-9, 10)
    ints = np.stack(np.meshgrid(r, r, r, indexing="ij"), axis=-1).reshape(-1, 3)
    G = _sorted_g(ints, wl.cell.lat)[:n_g]
    w = np.linspace(0.0, 40.0, 301)
    out = []
    for direct in (False, True):
        c = Context(0)
        if direct:
            c.set_memory_limit(1 << 40)
        set_inputs(c, wl)
        out.append(c.loss_diag(G, w, wl.eta_eV, "fp64").cpu().numpy())
        c.sync()
        c.close()
    assert np.max(np.abs(out[0] - out[1])) <= 1e-10 * np.max(np.abs(out[1]))
    assert not np.array_equal(out[0], out[1])
