"""Inversions beyond 128 G, where a matrix is shared by several workgroups:
the two forms of each size class on either side of the count at which the
dispatch changes, sizes at the edges of the 16- and 32-column tiles, and the
caller's storage (matrices untouched, a diagonal that overlaps them)."""
import numpy as np
import pytest

from paper_2603_12326_amd import Context

pytestmark = pytest.mark.gpu

# (n_G, n_w): few and many matrices of each class
_CASES = [(129, 129), (160, 130), (193, 129), (224, 140), (257, 129), (289, 129), (321, 129), (352, 3),
          (512, 130), (513, 65), (545, 64), (768, 65), (769, 33), (801, 32), (1024, 33)]


def _matrices(n, n_w, seed):
    import torch

    g = torch.Generator("cuda").manual_seed(seed)
    e = torch.randn((n_w, n, n), dtype=torch.complex128, device="cuda", generator=g) / n ** 0.5
    e[0, 0, 0] = 0.0  # the first pivot comes from another row
    return e


@pytest.mark.parametrize("n,n_w", _CASES)
def test_tiled_inverse(n, n_w):
    """diag(eps^-1) of matrices that need row exchanges against numpy's
    inverse (FP64, on the CPU) for the first, a middle and the last matrix.
    Bar 1e-10 normwise: unit roundoff times the condition number (up to a few
    thousand for such matrices) times n."""
    import torch

    c = Context(0)
    e = _matrices(n, n_w, 7 + n)
    keep = e.clone()
    diag = torch.empty((n_w, n), dtype=torch.complex128, device="cuda")
    loss = torch.empty((n_w, n), dtype=torch.float64, device="cuda")
    c.eps_inv_given(e, True, loss_out=loss, diag_out=diag)
    c.sync()
    assert torch.equal(e, keep)
    got = diag.cpu().numpy()
    for i in (0, n_w // 2, n_w - 1):
        ref = np.diagonal(np.linalg.inv(keep[i].cpu().numpy()))
        assert np.max(np.abs(got[i] - ref)) < 1e-10 * np.max(np.abs(ref)), (n, n_w, i)
    assert np.array_equal(loss.cpu().numpy(), -got.imag)


@pytest.mark.parametrize("n", [50, 128, 140])
def test_diagonal_over_its_matrices(n):
    """diag_out inside the storage of eps gives what separate storage gives."""
    import torch

    c = Context(0)
    e = _matrices(n, 5, n)
    diag = torch.empty((5, n), dtype=torch.complex128, device="cuda")
    c.eps_inv_given(e, True, diag_out=diag)
    c.sync()
    over = e.view(-1)[n:6 * n].view(5, n)
    c.eps_inv_given(e, True, diag_out=over)
    c.sync()
    assert torch.equal(over, diag)


@pytest.mark.parametrize("n,n_w", [(140, 4), (140, 130), (600, 66)])
def test_singular_matrix_is_named(n, n_w):
    """A zero column in one matrix reports that frequency and no other."""
    from paper_2603_12326_amd import QcxError

    c = Context(0)
    e = _matrices(n, n_w, 3)
    e[n_w - 2, :, n // 2] = 0.0
    c.eps_inv_given(e, True)
    with pytest.raises(QcxError, match=f"frequency index {n_w - 2}"):
        c.sync()
