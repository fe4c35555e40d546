"""qcx_eps_inv_given_noalloc runs its frequencies in chunks of 64 MiB; its
results are qcx_eps_inv_given's to the bit, also where the number of matrices
decides which kernels invert them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_w", [(100, 300), (150, 130), (190, 300), (259, 200), (320, 170), (400, 100), (400, 300),
                                   (512, 220), (600, 160), (768, 100), (900, 60), (1024, 40)])
def test_same_bits(n, n_w):
    import torch

    from paper_2603_12326_amd import Context

    g = torch.Generator(device="cuda").manual_seed(n)
    eps = torch.randn((n_w, n, n), dtype=torch.complex128, device="cuda", generator=g) * (0.4 / n**0.5)
    eps.diagonal(dim1=1, dim2=2).add_(1.5 + 0.3j)
    c = Context(0)
    out = []
    for noalloc in (False, True):
        diag = torch.zeros((n_w, n), dtype=torch.complex128, device="cuda")
        loss = torch.zeros((n_w, n), dtype=torch.float64, device="cuda")
        if noalloc:
            status = torch.zeros(1, dtype=torch.int32, device="cuda")
            c.eps_inv_given_noalloc(eps, True, loss, status, diag_out=diag)
            assert int(status) == 2**31 - 1
        else:
            c.eps_inv_given(eps, True, loss, diag_out=diag)
        c.sync()
        out.append((loss, diag))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    ref = torch.linalg.inv(eps[n_w // 2]).diagonal()
    assert float((out[0][1][n_w // 2] - ref).abs().max()) <= 1e-11 * float(ref.abs().max())
    c.close()
