"""An untrained network needs its fallback handle at create only: its values
and gradients do not read the handle, which may be closed before it."""
import numpy as np
import pytest

from paper_1011_4687_amd import synth

pytestmark = pytest.mark.gpu


def test_network_outlives_its_fallback():
    import torch
    from paper_1011_4687_amd.envpot import Environment, Surrogate, fourier_matrix, init_params
    print("[surrogate] fallback closed first", flush=True)
    E = Environment.from_synth(synth.make_tiny(1), precision="fp32c", neutralize=True)
    S = Surrogate(E, fourier_matrix(2, 0.25), init_params(2), radius=8.0, sigma=0.5)
    x = torch.from_numpy(synth.points_in_ball(np.random.default_rng(4), 3000, 8.0)).cuda()
    t = torch.zeros(3000, dtype=torch.float32, device="cuda")
    v, (loss, g) = S.predict(x).cpu().numpy(), S.loss_grad(x, t)
    E.close()
    others = [Environment.from_synth(synth.make_tiny(k), precision="fp64") for k in range(2, 8)]
    w, (loss2, g2) = S.predict(x).cpu().numpy(), S.loss_grad(x, t)
    assert np.array_equal(v, w)
    assert loss == loss2 and np.array_equal(g, g2)
    for e in others:
        e.close()
    S.close()
