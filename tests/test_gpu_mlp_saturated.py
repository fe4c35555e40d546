"""The networks where pre-activations are far below zero: SiLU is zero there,
however far."""
import numpy as np
import pytest

from oracle import mlp as ref
from synth.surrogate import mlp_init

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bias", [-70.0, -85.0, -1e4, -3e33, -1e38])
@pytest.mark.parametrize("layer", [0, 1, 3])
def test_far_negative(layer, bias):
    """Every third neuron of a hidden layer at `bias`: it contributes nothing
    (|SiLU(-70)| < 1e-28), as in the FP64 network with the same bf16 roundings.
    Bar: as for the fused forward pass, 2e-3 of the largest output."""
    import torch

    from paper_2603_12326_amd import Context, Mlp

    theta = mlp_init(31).copy()
    o = 0
    for i in range(5):
        a, b = ref.WIDTHS[i], ref.WIDTHS[i + 1]
        if i == layer:
            theta[o + a * b:o + a * b + b:3] = bias
        o += a * b + b
    x = np.random.default_rng(2).uniform(-1, 1, size=(300, ref.N_IN)).astype(np.float32)
    want, _ = ref.forward(theta.astype(np.float64), x.astype(np.float64), bf16=True)
    assert np.all(np.isfinite(want))
    c = Context(0)
    m = Mlp(c, 1)
    m.set_params(0, theta)
    y = torch.empty(len(x), dtype=torch.float32, device="cuda")
    m.forward(0, torch.from_numpy(x).cuda(), y)
    got = y.cpu().numpy()
    m.close()
    c.close()
    off = np.abs(got - want) >= 2e-3 * np.max(np.abs(want))
    assert np.mean(off) <= 0.01
    assert np.max(np.abs(got - want)) <= 2e-2 * np.max(np.abs(want))
