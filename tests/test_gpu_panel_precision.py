"""chi0 through energy panels where one row of densities spans orders of
magnitude: tight core shells whose densities stay of order 0.1 at the listed G
beside diffuse valence shells whose densities have fallen to 1e-2 .. 1e-4
there, with the core 100 to 1800 eV away.  The absorptive part below 30 eV,
which is the loss, comes from the small densities, or, below the gap, from the
tails of the weights alone."""
import numpy as np
import pytest

from synth.generator import (Basis, _sorted_g, bloch_overlap, fcc_cell, gamma_grid, lowdin, real_space_overlaps,
                             reciprocal_rows)

pytestmark = pytest.mark.gpu

# Of sqrt(max_w A_GG max_w A_G'G'), A the absorptive part.  FP32: operands of
# 2^-24 each and FP32 sums of at most 1024 steps of 16 transitions, whose
# rounding walks to at most sqrt(16384) 2^-24 = 7.6e-6.  Split-BF16: as much,
# and 2^-17 for each of the two bf16 pairs of a product.
_BAR = dict(fp32=8e-6, split_bf16=2.5e-5)


@pytest.fixture(scope="module")
def spread():
    cell = fcc_cell(10.26)
    shells = [(0, 400.0), (0, 0.3), (1, 30.0), (1, 0.25)]
    sa, sl, se = zip(*[(a, l, e) for a in (0, 1) for l, e in shells])
    basis = Basis(np.array(sa, np.int32), np.array(sl, np.int32), np.array(se))
    # the AOs themselves, orthonormalised: tight s, diffuse s | diffuse p, tight p
    order = [0, 8, 1, 9] + [a + i for a in (0, 8) for i in (5, 6, 7)] + [a + i for a in (0, 8) for i in (2, 3, 4)]
    kf = gamma_grid(7)
    q = np.array([0.3 * 2 * np.pi / cell.a, 0.02, 0.01])
    tn, s_t = real_space_overlaps(cell, basis)
    rng = np.random.default_rng(3)
    st = []
    for f in (kf, kf + (cell.lat @ q / (2 * np.pi))[None]):
        C = np.stack([lowdin(np.eye(16, dtype=complex), s)[:, order] for s in bloch_overlap(s_t, tn, f)])
        E = np.concatenate([rng.uniform(lo, hi, (len(f), n)) for n, lo, hi in
                            ((2, -1800.0, -100.0), (2, -12.0, 0.0), (6, 1.1, 15.0), (6, 50.0, 100.0))], 1)
        st += [np.ascontiguousarray(C), E]
    r = np.arange(-12, 13)
    g = _sorted_g(np.stack(np.meshgrid(r, r, r, indexing="ij"), -1).reshape(-1, 3), cell.lat)
    n = np.linalg.norm(g @ reciprocal_rows(cell.lat), axis=1)

    def rows(lo, hi):
        s = g[(n > lo) & (n < hi)]
        return np.concatenate([g[:1], s[np.linspace(0, len(s) - 1, 47).astype(int)]]).astype(np.int32)

    return cell, basis, kf, q, st, rows


def _absorptive(spread, G, w, eta, precision, direct):
    import torch

    from paper_2603_12326_amd import Context

    cell, basis, kf, q, st, _ = spread
    c = Context(0)
    if direct:
        c.set_memory_limit(1 << 40)
    c.set_cell_basis(cell.lat, cell.xyz, basis.shell_atom, basis.shell_l, basis.shell_exp, 1, 1)
    c.set_states(q, kf, 4, *st)
    c.pair_density(G)
    chi = torch.empty((len(w), len(G), len(G)), dtype=torch.complex128, device="cuda")
    c.chi0(w, eta, precision, True, chi)
    c.sync()
    panels = c.bulk_config()["stages"] == 0
    c.close()
    x = chi.cpu().numpy()
    return (x - np.conj(np.swapaxes(x, 1, 2))) / 2j, panels


@pytest.mark.parametrize("precision", ["fp32", "split_bf16"])
@pytest.mark.parametrize("eta,w_max", [(0.1, 30.0), (0.003, 1.0)])
@pytest.mark.parametrize("g_lo,g_hi", [(2.5, 3.0), (3.5, 4.0), (4.2, 4.6)])
def test_absorptive_part(spread, g_lo, g_hi, eta, w_max, precision):
    G, w = spread[-1](g_lo, g_hi), np.linspace(0.0, w_max, 300)
    ref, _ = _absorptive(spread, G, w, eta, "fp64", True)
    got, panels = _absorptive(spread, G, w, eta, precision, False)
    assert panels
    d = np.sqrt(np.max(np.abs(np.einsum("wgg->wg", ref)), axis=0))
    err = np.max(np.abs(got - ref) / (d[:, None] * d))
    print(f"{precision}: {err:.2e}")
    assert err <= _BAR[precision]


@pytest.mark.parametrize("precision", ["fp32", "split_bf16"])
@pytest.mark.parametrize("name", ["all_electron", "long_entries"])
def test_against_fp64(name, precision):
    """The all-electron basis (52 AOs, core levels to -1800 eV), and 170,368
    transitions, whose entries are longer than their usual 1,024: both modes
    within 1e-6 of the largest |chi0|, 16 units of their 24-bit operands."""
    import torch

    from paper_2603_12326_amd import Context
    from synth import make_all_electron, make_si_ng113
    from tests.gpu_helpers import set_inputs

    if name == "all_electron":
        wl, n_g, w = make_all_electron(n_w=200, kgrid=4), 97, np.linspace(0.0, 100.0, 200)
    else:
        wl, n_g, w = make_si_ng113(n_q=1, kgrid=11), 61, np.linspace(0.0, 60.0, 300)
    chi = []
    for direct in (True, False):
        c = Context(0)
        if direct:
            c.set_memory_limit(1 << 42)
        set_inputs(c, wl)
        c.pair_density(wl.G_int[:n_g])
        x = torch.empty((len(w), n_g, n_g), dtype=torch.complex128, device="cuda")
        c.chi0(w, 0.1, "fp64" if direct else precision, True, x)
        c.sync()
        assert direct or c.bulk_config()["stages"] == 0
        c.close()
        chi.append(x)
    err = float((chi[1] - chi[0]).abs().max() / chi[0].abs().max())
    print(f"{name} {precision}: {err:.2e}")
    assert err <= 1e-6
