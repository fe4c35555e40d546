"""Cases for timing the library through its public entry points.

Each case is one call (or the few calls that belong together) as a program
that computes loss functions makes it, with synthetic states of the sizes this
repository uses: diamond-structure cells, Gaussian shells, k grids of 4^3 to
10^3 points, 27 to 749 G vectors, tens to hundreds of frequencies.  Random
coefficients are smooth in k and orthonormalised with the overlap of the
Gaussians; band energies are uniform in a valence and a conduction range.

The bulk of chi0 in FP32 or split-BF16 carries single precision at most, and
the order of its sums follows a choice made by timing, so it differs from one
process to the next; a program that asked for it keeps its tables in single
precision, and so do these cases.  FP64 results stay in double precision.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2603_12326_amd import qcx

HA = 27.211386245988
DEV = "cuda"

# per atom: (angular momentum, exponent)
SHELLS = {
    # two s and one p shell: 10 AOs for two atoms
    "small": [(0, 0.5), (0, 2.0), (1, 0.8)],
    # three s, two p and one d shell: 28 AOs
    "spd": [(0, 12.0), (0, 1.4), (0, 0.2), (1, 1.6), (1, 0.25), (2, 0.6)],
    # core shells as in an all-electron calculation: 52 AOs
    "core": [(0, 6000.0), (0, 900.0), (0, 120.0), (0, 18.0), (0, 2.0), (0, 0.25),
             (1, 40.0), (1, 9.0), (1, 2.2), (1, 0.7), (1, 0.25), (2, 0.6)],
}
# (occupied groups, empty groups) of (bands, lowest, highest energy in eV)
BANDS = {
    "small": ([(4, -12.0, 0.0)], [(6, 1.1, 15.0)]),
    "spd": ([(4, -12.0, 0.0)], [(16, 1.1, 15.0)]),
    "core": ([(5, -1800.0, -100.0), (4, -12.0, 0.0)], [(28, 1.1, 100.0)]),
}
CELLS = [6.74, 10.26, 10.69, 10.68, 8.24]       # lattice constants (bohr) of the mixed batch


# ------------------------------------------------------------------ crystal
def _cell(a):
    lat = 0.5 * a * np.array([[0.0, 1.0, 1.0], [1.0, 0.0, 1.0], [1.0, 1.0, 0.0]])
    return lat, np.array([[0.0, 0.0, 0.0], [0.25 * a, 0.25 * a, 0.25 * a]])


def _basis(name):
    sh = SHELLS[name]
    return ([ia for ia in (0, 1) for _ in sh], [l for _ in (0, 1) for l, _ in sh],
            [e for _ in (0, 1) for _, e in sh])


def _g_list(lat, n):
    m = 4
    while (2 * m + 1) ** 3 < 4 * n:
        m += 1
    r = np.arange(-m, m + 1)
    g = np.stack(np.meshgrid(r, r, r, indexing="ij"), -1).reshape(-1, 3)
    g2 = np.round(np.sum((g @ (2 * math.pi * np.linalg.inv(lat).T)) ** 2, 1), 9)
    return np.ascontiguousarray(g[np.lexsort((g[:, 2], g[:, 1], g[:, 0], g2))][:n].astype(np.int32))


def _k_grid(n):
    m = np.arange(n) / n
    return np.stack(np.meshgrid(m, m, m, indexing="ij"), -1).reshape(-1, 3)


CELL_N = np.stack(np.meshgrid(*[np.arange(-1, 2)] * 3, indexing="ij"), -1).reshape(-1, 3)


def _ao_terms(l, e):
    """Monomials (coefficient, powers) of each function of a shell, unit norm."""
    g = (2 * e / math.pi) ** 0.75
    if l == 0:
        return [[(g, (0, 0, 0))]]
    if l == 1:
        c = g * math.sqrt(4 * e)
        return [[(c, (1, 0, 0))], [(c, (0, 1, 0))], [(c, (0, 0, 1))]]
    d = 4 * e * g
    h = d / (2 * math.sqrt(3.0))
    return [[(d, (1, 1, 0))], [(d, (0, 1, 1))],
            [(2 * h, (0, 0, 2)), (-h, (2, 0, 0)), (-h, (0, 2, 0))],
            [(d, (1, 0, 1))], [(0.5 * d, (2, 0, 0)), (-0.5 * d, (0, 2, 0))]]


def _integrals(lat, xyz, basis, Q):
    """F[cell][Q][mu][nu] = int chi_mu(r) e^{iQr} chi_nu(r - T) d^3r, complex128 on the GPU.

    Per axis the product of two Gaussians is one Gaussian about P; with the
    plane wave folded into a shift of the centre by iQ/2p, three Gauss-Hermite
    points integrate the polynomials (degree at most four) exactly."""
    at, ls, ex = basis
    Q = torch.as_tensor(np.asarray(Q, np.float64), device=DEV)
    T = torch.as_tensor(CELL_N @ lat, device=DEV)
    A = torch.as_tensor(xyz[at], device=DEV)
    e = torch.as_tensor(np.array(ex), device=DEV)
    a, b = e[:, None, None], e[None, :, None]
    p = a + b
    nodes, wts = np.polynomial.hermite.hermgauss(3)
    J = []
    for x in range(3):
        ca, cb = A[:, x][:, None, None], A[:, x][None, :, None] + T[:, x][None, None, :]
        P = (a * ca + b * cb) / p
        pre = torch.exp(-a * b / p * (ca - cb) ** 2) / torch.sqrt(p)
        q = Q[:, x]
        ph = torch.exp(1j * P[..., None] * q - q * q / (4 * p[..., None])) * pre[..., None]
        sh = 1j * q / (2 * p[..., None])
        tab = [[0] * 3 for _ in range(3)]
        for t, w in zip(nodes, wts):
            u = t / torch.sqrt(p)[..., None] + sh
            va, vb = u + (P - ca)[..., None], u + (P - cb)[..., None]
            pa, pb = [w * ph, w * ph * va, w * ph * va * va], [1.0, vb, vb * vb]
            for i in range(3):
                for j in range(3):
                    tab[i][j] = tab[i][j] + pa[i] * pb[j]
        J.append(tab)
    aos = [(s, t) for s in range(len(ls)) for t in _ao_terms(ls[s], ex[s])]
    n = len(aos)
    F = torch.empty((len(T), len(Q), n, n), dtype=torch.complex128, device=DEV)
    for m, (s, tm) in enumerate(aos):
        for v, (r, tv) in enumerate(aos):
            acc = 0
            for cm, i in tm:
                for cv, j in tv:
                    acc = acc + cm * cv * (J[0][i[0]][j[0]][s, r] * J[1][i[1]][j[1]][s, r] *
                                           J[2][i[2]][j[2]][s, r])
            F[:, :, m, v] = acc
    return F


_OVERLAPS = {}


def _overlaps(a, name):
    """Overlap integrals of one cell and basis (the same for every seed)."""
    if (a, name) not in _OVERLAPS:
        lat, xyz = _cell(a)
        _OVERLAPS[a, name] = _integrals(lat, xyz, _basis(name), np.zeros((1, 3)))[:, 0].cpu().numpy()
    return _OVERLAPS[a, name]


def _states(a, name, kgrid, q, rng):
    """Orthonormal coefficients smooth in k, and energies, at k and at k + q."""
    lat, _ = _cell(a)
    F0 = _overlaps(a, name)
    occ, emp = BANDS[name]
    n_occ, n_b = sum(g[0] for g in occ), sum(g[0] for g in occ + emp)
    nao = F0.shape[-1]
    kf = _k_grid(kgrid)
    harm = np.vstack([np.zeros((1, 3)), np.eye(3), -np.eye(3)])
    X = rng.standard_normal((7, nao, n_b)) + 1j * rng.standard_normal((7, nao, n_b))
    X[1:] *= 0.35
    out = []
    for f in (kf, kf + lat @ q / (2 * math.pi)):
        S = (np.exp(2j * math.pi * (f @ CELL_N.T)) @ F0.reshape(len(CELL_N), -1)).reshape(-1, nao, nao)
        C = (np.exp(2j * math.pi * (f @ harm.T)) @ X.reshape(7, -1)).reshape(-1, nao, n_b)
        for _ in range(2):
            L = np.linalg.cholesky(np.conj(np.swapaxes(C, 1, 2)) @ (S @ C))
            C = np.conj(np.swapaxes(np.linalg.solve(L, np.conj(np.swapaxes(C, 1, 2))), 1, 2))
        E = np.concatenate([np.sort(rng.uniform(lo, hi, (len(f), c)), 1) for c, lo, hi in occ + emp], 1)
        out += [np.ascontiguousarray(C), E]
    return kf, n_occ, out


def _problem(case, seed, q_frac=0.3):
    lat, xyz = _cell(case["a"])
    q = np.array([q_frac * 2 * math.pi / case["a"], 0.0, 0.0])
    kf, n_occ, st = _states(case["a"], case["basis"], case["kgrid"], q, np.random.default_rng(seed))
    return dict(lat=lat, xyz=xyz, basis=_basis(case["basis"]), q=q, kf=kf, n_occ=n_occ, st=st,
                G=_g_list(lat, case["n_g"]))


def _w(case):
    return np.linspace(0.0, case["w_max"], case["n_w"])


def _put(x):
    return torch.as_tensor(x, device=DEV)


def _context(pb, G=None):
    """A context with the states set from device memory (and the pair densities)."""
    c = qcx.Context(0)
    at, ls, ex = pb["basis"]
    c.set_cell_basis(pb["lat"], pb["xyz"], at, ls, ex)
    dev = [_put(pb["kf"])] + [_put(x) for x in pb["st"]]
    c.set_states(pb["q"], dev[0], pb["n_occ"], *dev[1:])
    if G is not None:
        c.pair_density(G)
    return c, dev


# ------------------------------------------------------- 64-bit references
def _densities(pb, G):
    """R[t][G] with t = (side, k, v, c), complex128 on the GPU."""
    Ck, _, Cq, _ = [_put(x) for x in pb["st"]]
    no, nk = pb["n_occ"], len(pb["kf"])
    nc = Ck.shape[2] - no
    Q = pb["q"] + G @ (2 * math.pi * np.linalg.inv(pb["lat"]).T)
    ph = _put(np.exp(2j * math.pi * (pb["kf"] @ CELL_N.T)))
    CqH = Cq.conj().transpose(1, 2).contiguous()
    R = torch.empty((2, nk, no, nc, len(G)), dtype=torch.complex128, device=DEV)
    for g0 in range(0, len(G), 128):
        F = _integrals(pb["lat"], pb["xyz"], pb["basis"], Q[g0:g0 + 128])
        for g in range(F.shape[1]):
            M = (ph @ F[:, g].reshape(len(CELL_N), -1)).reshape(nk, F.shape[2], F.shape[3])
            B = torch.matmul(CqH, torch.matmul(M, Ck))
            R[0, ..., g0 + g] = B[:, no:, :no].transpose(1, 2)
            R[1, ..., g0 + g] = B[:, :no, no:]
    return R.reshape(-1, len(G))


def _energies(pb):
    _, ek, _, eq = [x / HA for x in pb["st"]]
    no = pb["n_occ"]
    return ((eq[:, None, no:] - ek[:, :no, None]).reshape(-1),
            (ek[:, None, no:] - eq[:, :no, None]).reshape(-1))


def _norm(pb):
    return 2.0 / (len(pb["kf"]) * abs(np.linalg.det(pb["lat"])))


def _weights(pb, w, eta):
    """Per frequency the weight of every transition in the response."""
    dr, da = [_put(x) for x in _energies(pb)]
    for x in w / HA:
        yield _norm(pb) * torch.cat([1 / (x - dr + 1j * eta / HA), -1 / (x + da - 1j * eta / HA)])


def _hat(z):
    """int (1 - |y|) / (z - y) dy over [-1, 1], in extended precision."""
    z = np.asarray(z, np.clongdouble)
    f = lambda u: u * np.log(u)  # noqa: E731
    return (f(z + 1) - 2 * f(z) + f(z - 1)).astype(np.complex128)


def _weights_binned(pb, w, eta, width):
    """As _weights, every transition shared between the two nearest bins."""
    d = width / HA
    for i in range(0, len(w), 64):
        rows = []
        for E, s in zip(_energies(pb), (1.0, -1.0)):
            b0 = int(np.floor(E.min() / d))
            c = np.arange(b0, int(np.floor(E.max() / d)) + 2)
            K = s * _hat((w[i:i + 64, None] / HA - s * c * d) / d + 1j * s * eta / HA / d) / d
            u = E / d
            j = np.floor(u).astype(np.int64)
            x, j, K = _put(u - j), _put(j - b0), _put(K)
            rows.append(K[:, j] * (1 - x) + K[:, j + 1] * x)
        yield from _norm(pb) * torch.cat(rows, 1)


def _chi0(R, weights):
    RH = R.conj().T.contiguous()
    return torch.stack([torch.matmul(RH, R * x[:, None]) for x in weights])


def _vq(pb, G):
    Q = pb["q"] + G @ (2 * math.pi * np.linalg.inv(pb["lat"]).T)
    return _put(math.sqrt(4 * math.pi) / np.linalg.norm(Q, axis=1))


def _inverse_diagonal(eps):
    e = eps.cpu().numpy()
    return np.stack([np.diagonal(np.linalg.inv(m)) for m in e])


def _exact_loss(pb, G, w, eta):
    v = _vq(pb, G)
    eps = torch.eye(len(G), device=DEV) - v[:, None] * _chi0(_densities(pb, G), _weights(pb, w, eta)) * v
    return _inverse_diagonal(eps)


def _single(case, x):
    """Tables of a reduced-precision bulk are kept in single precision."""
    if case["precision"] == "fp64":
        return x
    return x.to(torch.complex64 if x.is_complex() else torch.float32)


# ------------------------------------------------------------------- kinds
class _QPoint:
    """One momentum from its states to the loss: states, pair densities,
    chi0, the inverse of eps and the loss, as the loop over q runs them."""

    @staticmethod
    def prepare(case, seed):
        pb = _problem(case, seed)
        c, dev = _context(pb)
        n = (case["n_w"], case["n_g"])
        return dict(c=c, dev=dev, pb=pb, w=_w(case), case=case,
                    diag=torch.empty(n, dtype=torch.complex128, device=DEV),
                    loss=torch.empty(n, dtype=torch.float64, device=DEV))

    @staticmethod
    def run(s):
        c, pb, dev, case = s["c"], s["pb"], s["dev"], s["case"]
        c.set_states(pb["q"], dev[0], pb["n_occ"], *dev[1:])
        c.pair_density(pb["G"])
        c.chi0(s["w"], case["eta"], case["precision"])
        c.eps_inv(True, s["diag"])
        c.loss(s["loss"])
        return {"loss": _single(case, s["loss"]), "diag": _single(case, s["diag"])}

    @staticmethod
    def exact(case, seed):
        pb = _problem(case, seed)
        d = _exact_loss(pb, pb["G"], _w(case), case["eta"])
        return {"loss": -d.imag, "diag": d}


class _Density:
    """The pair densities of one momentum, kept by the caller."""

    @staticmethod
    def prepare(case, seed):
        pb = _problem(case, seed)
        c, dev = _context(pb)
        nk, nc = len(pb["kf"]), pb["st"][0].shape[2] - pb["n_occ"]
        return dict(c=c, dev=dev, pb=pb,
                    rho=torch.empty((2, nk, pb["n_occ"], nc, case["n_g"]), dtype=torch.complex128, device=DEV))

    @staticmethod
    def run(s):
        s["c"].pair_density(s["pb"]["G"], s["rho"])
        return s["rho"]

    @staticmethod
    def exact(case, seed):
        pb = _problem(case, seed)
        nk, nc = len(pb["kf"]), pb["st"][0].shape[2] - pb["n_occ"]
        return _densities(pb, pb["G"]).reshape(2, nk, pb["n_occ"], nc, -1)


class _Chi0:
    """chi0 from pair densities at hand (direct, or through the binned
    spectral part when the case gives a bin width)."""

    @staticmethod
    def prepare(case, seed):
        pb = _problem(case, seed)
        c, dev = _context(pb, _g_list(pb["lat"], case["n_g"]))
        return dict(c=c, dev=dev, w=_w(case), case=case,
                    chi=torch.empty((case["n_w"], case["n_g"], case["n_g"]), dtype=torch.complex128, device=DEV))

    @staticmethod
    def run(s):
        case = s["case"]
        if case.get("bin"):
            s["c"].chi0_kk(s["w"], case["eta"], case["bin"], s["chi"])
        else:
            s["c"].chi0(s["w"], case["eta"], case["precision"], True, s["chi"])
        return _single(case, s["chi"])

    @staticmethod
    def exact(case, seed):
        pb = _problem(case, seed)
        if case.get("bin"):
            ws = _weights_binned(pb, _w(case), case["eta"], case["bin"])
        else:
            ws = _weights(pb, _w(case), case["eta"])
        return _chi0(_densities(pb, pb["G"]), ws)


class _Inverse:
    """diag(eps^-1) and the loss of dielectric matrices formed elsewhere."""

    @staticmethod
    def prepare(case, seed):
        g = torch.Generator(device=DEV).manual_seed(seed)
        n_w, n = case["n_w"], case["n_g"]
        eps = torch.randn((n_w, n, n), dtype=torch.complex128, device=DEV, generator=g) * (0.4 / math.sqrt(n))
        d = torch.rand((n_w, n), dtype=torch.float64, device=DEV, generator=g)
        eps.diagonal(dim1=1, dim2=2).add_(torch.complex(1.2 + 2 * d, 0.3 + d))
        return dict(c=qcx.Context(0), eps=eps, diag=torch.empty((n_w, n), dtype=torch.complex128, device=DEV),
                    loss=torch.empty((n_w, n), dtype=torch.float64, device=DEV))

    @staticmethod
    def run(s):
        s["c"].eps_inv_given(s["eps"], True, s["loss"], s["diag"])
        return {"loss": s["loss"], "diag": s["diag"]}

    @staticmethod
    def exact(case, seed):
        d = _inverse_diagonal(_Inverse.prepare(case, seed)["eps"])
        return {"loss": -d.imag, "diag": d}


class _Diagonal:
    """Loss without local fields for a long G list (the high-momentum part
    of the composite dielectric function)."""

    @staticmethod
    def prepare(case, seed):
        pb = _problem(case, seed)
        c, dev = _context(pb)
        n = (case["n_w"], case["n_g"])
        return dict(c=c, dev=dev, G=pb["G"], w=_w(case), case=case,
                    loss=torch.empty(n, dtype=torch.float64, device=DEV),
                    inv=torch.empty(n, dtype=torch.complex128, device=DEV))

    @staticmethod
    def run(s):
        case = s["case"]
        s["c"].loss_diag(s["G"], s["w"], case["eta"], case["precision"], s["loss"], s["inv"])
        return {"loss": _single(case, s["loss"]), "inv": _single(case, s["inv"])}

    @staticmethod
    def exact(case, seed):
        pb = _problem(case, seed)
        W = torch.stack(list(_weights(pb, _w(case), case["eta"])))
        inv = []
        for g0 in range(0, case["n_g"], 512):
            G = pb["G"][g0:g0 + 512]
            R = _densities(pb, G)
            r2 = (R.real ** 2 + R.imag ** 2).to(torch.complex128)
            inv.append(1 / (1 - _vq(pb, G) ** 2 * torch.matmul(W, r2)))
        inv = torch.cat(inv, 1)
        return {"loss": -inv.imag, "inv": inv}


class _Batch:
    """Uneven items (cells, k grids, N_G, frequency lists) in one call, the
    pair densities inside it."""

    @staticmethod
    def items(case):
        out = []
        for i in range(case["items"]):
            j = i + case["first"]
            out.append(dict(a=CELLS[j % 5], basis="small", kgrid=6 + (3 * j) % 5, n_g=[59, 113, 181, 259][j % 4],
                            n_w=5 + (case["step_w"] * j) % 200, w_max=60.0, eta=0.1, q=0.1 + 0.04 * (j % 20)))
        return out

    @staticmethod
    def prepare(case, seed):
        s = dict(ctxs=[], keep=[], G=[], items=[], case=case)
        for i, it in enumerate(_Batch.items(case)):
            pb = _problem(it, seed + 1000 * i, it["q"])
            c, dev = _context(pb)
            s["ctxs"].append(c)
            s["keep"].append(dev)
            s["G"].append(pb["G"])
            s["items"].append(dict(ctx=i, w_eV=_w(it), eta_eV=it["eta"],
                                   loss_out=torch.empty((it["n_w"], it["n_g"]), dtype=torch.float64, device=DEV)))
        return s

    @staticmethod
    def run(s):
        qcx.run_batch(s["ctxs"], s["items"], s["case"]["precision"], G_lists=s["G"])
        return [_single(s["case"], it["loss_out"]) for it in s["items"]]

    @staticmethod
    def exact(case, seed):
        out = []
        for i, it in enumerate(_Batch.items(case)):
            pb = _problem(it, seed + 1000 * i, it["q"])
            out.append(-_exact_loss(pb, pb["G"], _w(it), it["eta"]).imag)
        return out


WIDTHS = [49, 256, 256, 256, 256, 1]


def _net(rng):
    parts = []
    for i in range(5):
        parts.append(rng.standard_normal(WIDTHS[i + 1] * WIDTHS[i]) * math.sqrt((1.0 if i == 4 else 2.0) / WIDTHS[i]))
        parts.append(np.zeros(WIDTHS[i + 1]))
    return np.concatenate(parts).astype(np.float32)


def _layers(theta):
    out, o = [], 0
    for i in range(5):
        n = WIDTHS[i + 1] * WIDTHS[i]
        out.append((theta[o:o + n].reshape(WIDTHS[i + 1], WIDTHS[i]), theta[o + n:o + n + WIDTHS[i + 1]]))
        o += n + WIDTHS[i + 1]
    return out


def _net_forward(layers, h):
    for i, (W, b) in enumerate(layers):
        h = torch.matmul(h, W.T.contiguous()) + b
        if i < 4:
            h = h * torch.sigmoid(h)
    return h[:, 0]


def _features(qw, q_max, w_max, lat):
    Q, w = qw[:, :3], qw[:, 3]
    n = Q.norm(dim=1)
    f = [2 * n / q_max - 1, *(Q / n[:, None]).T, 2 * w / w_max - 1]
    for x in (w / w_max, n / q_max):
        for j in range(8):
            f += [torch.sin(math.pi * 2 ** (j / 2) * x), torch.cos(math.pi * 2 ** (j / 2) * x)]
    for i in range(3):
        t = torch.matmul(Q, lat[i])
        for h in (1, 2):
            f += [torch.sin(h * t), torch.cos(h * t)]
    return torch.stack(f, 1)


class _Query:
    """The surrogate's answer and error estimate for a block of (Q, w)."""

    @staticmethod
    def prepare(case, seed):
        rng = np.random.default_rng(seed)
        lat, _ = _cell(10.26)
        c = qcx.Context(0)
        m = qcx.Mlp(c, case["members"])
        nets = [_net(rng) for _ in range(case["members"])]
        for i, p in enumerate(nets):
            m.set_params(i, p)
        m.set_encoding(4.0, 60.0, lat, -4.0, 2.0, 3.0)
        n = case["n"]
        qw = np.concatenate([rng.uniform(-2.0, 2.0, (n, 3)), rng.uniform(0.0, 60.0, (n, 1))], 1)
        out = lambda: torch.empty(n, dtype=torch.float64, device=DEV)  # noqa: E731
        return dict(c=c, m=m, nets=nets, lat=lat, qw=_put(qw), loss=out(), err=out())

    @staticmethod
    def run(s):
        s["m"].query(s["qw"], s["loss"], s["err"])
        # the networks' products are bf16 with FP32 sums
        return {"loss": s["loss"].to(torch.float32), "err": s["err"].to(torch.float32)}

    @staticmethod
    def exact(case, seed):
        s = _Query.prepare(case, seed)
        x = _features(s["qw"], 4.0, 60.0, _put(s["lat"]))
        y = torch.stack([_net_forward(_layers(_put(p.astype(np.float64))), x) for p in s["nets"]])
        return {"loss": torch.exp(-4.0 + 2.0 * y.mean(0)), "err": 3.0 * 2.0 * y.std(0)}


class _Train:
    """A few Adam steps of one network from its initial weights."""

    @staticmethod
    def prepare(case, seed):
        rng = np.random.default_rng(seed)
        lat, _ = _cell(10.26)
        n, b = case["n"], case["batch"]
        c = qcx.Context(0)
        qw = _put(np.concatenate([rng.uniform(-2.0, 2.0, (n, 3)), rng.uniform(0.0, 60.0, (n, 1))], 1))
        x = _features(qw, 4.0, 60.0, _put(lat)).to(torch.float32).contiguous()
        t = (torch.sin(qw[:, 3] / 6) * torch.cos(qw[:, :3].sum(1))).to(torch.float32)
        order = np.concatenate([rng.permutation(n) for _ in range(case["steps"] * b // n + 1)])
        return dict(c=c, m=qcx.Mlp(c, 1), theta=_net(rng), x=x, t=t, case=case,
                    order=_put(order[:case["steps"] * b].astype(np.int32)))

    @staticmethod
    def run(s):
        m = s["m"]
        m.set_params(0, s["theta"])
        hist = m.train(0, s["x"], s["t"], s["case"]["batch"], s["order"], 1e-3, 1e-5)
        return {"theta": m.get_params(0), "hist": hist}

    @staticmethod
    def exact(case, seed):
        s = _Train.prepare(case, seed)
        th = _put(s["theta"].astype(np.float64)).requires_grad_(True)
        m, v, hist = torch.zeros_like(th), torch.zeros_like(th), []
        x, t = s["x"].double(), s["t"].double()
        for k in range(case["steps"]):
            o = s["order"][k * case["batch"]:(k + 1) * case["batch"]].long()
            loss = ((_net_forward(_layers(th), x[o]) - t[o]) ** 2).mean()
            g, = torch.autograd.grad(loss, th)
            hist.append(float(loss))
            m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
            lr = 1e-5 + (1e-3 - 1e-5) * (1 + math.cos(math.pi * k / case["steps"])) / 2
            up = lr * (m / (1 - 0.9 ** (k + 1))) / ((v / (1 - 0.999 ** (k + 1))).sqrt() + 1e-8)
            th = (th - up).detach().requires_grad_(True)
        return {"theta": th.detach(), "hist": np.array(hist)}


KINDS = dict(q_point=_QPoint, density=_Density, chi0=_Chi0, inverse=_Inverse, diagonal=_Diagonal, batch=_Batch,
             query=_Query, train=_Train)


def prepare(case, seed):
    return dict(kind=case["kind"], s=KINDS[case["kind"]].prepare(case, seed))


def run(state):
    return KINDS[state["kind"]].run(state["s"])


def exact(case, seed):
    return KINDS[case["kind"]].exact(case, seed)


# -------------------------------------------------------------------- work
def _sizes(case):
    occ, emp = BANDS[case["basis"]]
    no, nc = sum(g[0] for g in occ), sum(g[0] for g in emp)
    nao = sum(2 * l + 1 for _, l in zip(*_basis(case["basis"])[:2]))
    return no, nc, nao, case["kgrid"] ** 3


def _density_work(case):
    """States in, densities out; the lattice sum once per AO pair, and the
    contraction with the valence bands first."""
    no, nc, nao, nk = _sizes(case)
    n_t = 2 * nk * no * nc
    flops = 8 * nk * case["n_g"] * (27 * nao * nao + 2 * nao * nao * no + 2 * nao * no * nc)
    return 2 * 16 * nk * nao * (no + nc), 16 * n_t * case["n_g"], n_t, flops


def work(case):
    k = case["kind"]
    if k == "inverse":
        n, n_w = case["n_g"], case["n_w"]
        return {"bytes": n_w * (16 * n * n + 24 * n), "flops": 8 * n_w * n ** 3}
    if k == "query":
        macs = sum(WIDTHS[i] * WIDTHS[i + 1] for i in range(5))
        return {"bytes": 48 * case["n"], "flops": 2 * macs * case["n"] * case["members"]}
    if k == "train":
        macs = sum(WIDTHS[i] * WIDTHS[i + 1] for i in range(5))
        rows = case["steps"] * case["batch"]
        return {"bytes": 200 * case["n"] + 4 * rows + 8 * 210433, "flops": 6 * macs * rows}
    if k == "batch":
        each = [work(dict(it, kind="q_point", precision=case["precision"])) for it in _Batch.items(case)]
        return {x: sum(e[x] for e in each) for x in ("bytes", "flops")}
    n_w, n = case.get("n_w", 0), case["n_g"]
    states, dens, n_t, f_rho = _density_work(case)
    if k == "density":
        return {"bytes": states + dens, "flops": f_rho}
    # every transition and G pair enters the response at least once, and every
    # frequency and pair is written at least once
    pairs = n if k == "diagonal" else n * (n + 1) // 2
    f_chi = 8 * n_t * pairs
    if k == "chi0":
        return {"bytes": dens + 16 * n_w * n * n, "flops": f_chi}
    if k == "diagonal":
        return {"bytes": states + 24 * n_w * n, "flops": f_rho + f_chi}
    return {"bytes": states + 24 * n_w * n, "flops": f_rho + f_chi + 8 * n_w * n ** 3}


# ------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest calculation here: one momentum, few bands, 27 G, FP64
        dict(name="q_small_fp64", kind="q_point", a=10.26, basis="small", kgrid=4, n_g=27, n_w=128, w_max=40.0,
             eta=0.2, precision="fp64"),
        # the benchmark's momentum: 65,536 transitions, 113 G, 400 frequencies
        dict(name="q_113_split", kind="q_point", a=10.26, basis="spd", kgrid=8, n_g=113, n_w=400, w_max=60.0,
             eta=0.1, precision="split_bf16"),
        # pair densities of the benchmark's momentum, for a caller that keeps them
        dict(name="density_113", kind="density", a=10.26, basis="spd", kgrid=8, n_g=113),
        # all-electron basis: core shells, nine occupied bands, the larger contraction
        dict(name="density_core", kind="density", a=10.26, basis="core", kgrid=4, n_g=181),
        # response in full double precision on a medium grid
        dict(name="chi0_fp64", kind="chi0", a=10.69, basis="spd", kgrid=6, n_g=89, n_w=150, w_max=50.0, eta=0.15,
             precision="fp64"),
        # single precision, a wider G set and a finer k grid of a small basis
        dict(name="chi0_fp32", kind="chi0", a=8.24, basis="small", kgrid=8, n_g=181, n_w=155, w_max=60.0, eta=0.1,
             precision="fp32"),
        # the spectral route at the benchmark's sizes
        dict(name="kk_113", kind="chi0", a=10.26, basis="spd", kgrid=8, n_g=113, n_w=400, w_max=60.0, eta=0.1,
             bin=0.025, precision="fp64"),
        # inverses of a mid-sized set, as one batch item or a caller with its own eps has them
        dict(name="inverse_259", kind="inverse", n_g=259, n_w=175),
        # the part of the composite dielectric function without local fields, over two chunks of G
        dict(name="diagonal_4500", kind="diagonal", a=10.26, basis="spd", kgrid=6, n_g=4500, n_w=400, w_max=60.0,
             eta=0.1, precision="split_bf16"),
        # uneven items of the mixed batch
        dict(name="batch_8", kind="batch", items=8, first=3, step_w=30, precision="split_bf16"),
        # a surrogate fit, and its answers for one block of a query grid
        dict(name="train_4096", kind="train", n=65536, batch=4096, steps=16),
        dict(name="query_100k", kind="query", n=100489, members=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["q_point", "density", "chi0", "chi0", "kk", "inverse", "diagonal", "batch", "train", "query"])
    if kind == "inverse":
        n = _log_int(rng, 9, 400)
        return dict(kind=kind, n_g=n, n_w=max(1, min(_log_int(rng, 8, 500), int(3e9 / n ** 3))))
    if kind == "train":
        b = _log_int(rng, 256, 4096)
        return dict(kind=kind, n=_log_int(rng, 8192, 65536), batch=b, steps=rng.randint(4, 16))
    if kind == "query":
        return dict(kind=kind, n=_log_int(rng, 500, 100000), members=rng.randint(2, 4))
    if kind == "batch":
        return dict(kind=kind, items=rng.randint(2, 6), first=rng.randint(0, 19), step_w=rng.randint(7, 60),
                    precision=rng.choice(["split_bf16", "fp32"]))
    basis = rng.choice(["small", "small", "spd"])
    c = dict(kind=kind, a=round(rng.uniform(6.7, 10.7), 2), basis=basis, kgrid=rng.randint(3, 8),
             n_g=_log_int(rng, 27, 113 if basis == "spd" else 181))
    if kind == "density":
        if rng.random() < 0.3:
            c.update(basis="core", kgrid=rng.randint(2, 4))
        return c
    c.update(n_w=_log_int(rng, 8, 400), w_max=round(rng.uniform(30.0, 60.0), 1), eta=round(rng.uniform(0.08, 0.3), 3))
    if kind == "kk":
        c.update(kind="chi0", bin=round(rng.uniform(0.02, 0.1), 3), precision="fp64")
    elif kind == "diagonal":
        c.update(kgrid=rng.randint(3, 6), n_g=_log_int(rng, 300, 4500), precision=rng.choice(["split_bf16", "split_bf16", "fp64"]))
    else:
        c.update(precision=rng.choice(["fp64", "fp32", "split_bf16", "split_bf16"]))
    return c
