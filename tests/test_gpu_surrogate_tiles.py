"""The network's kernels at the edges of their tiles (32 rows, two row blocks
of 32 for many rows, 128-row gradient partials) and of the baseline's degree.
The layers themselves are held against the oracle in test_gpu_surrogate.py;
here a row's result must not depend on where in a batch it stands."""
import numpy as np
import pytest

from paper_1011_4687_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fallback():
    from paper_1011_4687_amd.envpot import Environment
    return Environment.from_synth(synth.make_tiny(1), precision="fp32c", neutralize=True)


def _net(fallback, **kw):
    from paper_1011_4687_amd.envpot import Surrogate, fourier_matrix, init_params
    return Surrogate(fallback, fourier_matrix(2, 0.25), init_params(2), radius=8.0, **kw)


def _points(n, seed=9):
    return synth.points_in_ball(np.random.default_rng(seed), n, 8.0)


@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 64, 65, 127, 16385, 32705, 32767, 32768, 32769, 40001])
def test_predict_does_not_depend_on_the_tile(fallback, n):
    import torch
    print(f"[tiles] predict {n}", flush=True)
    S = _net(fallback, sigma=0.5)
    pts = _points(65600)
    # the first 1000 rows by themselves: one row block per tile
    head = S.predict(torch.from_numpy(pts[:1000]).cuda()).cpu().numpy()
    every = S.predict(torch.from_numpy(pts).cuda()).cpu().numpy()
    part = S.predict(torch.from_numpy(pts[-n:].copy()).cuda()).cpu().numpy()
    assert np.array_equal(every[:1000], head)
    assert np.array_equal(part, every[-n:])
    S.close()


@pytest.mark.parametrize("degree", range(9))
def test_baseline_of_every_degree(fallback, degree):
    """poly(r/R): at most 165 terms of products of up to eight factors, each
    rounded to 2^-53; the network's share (1e-6 of unit size) cancels."""
    import torch
    from oracle import mlp_oracle as M
    print(f"[tiles] baseline {degree}", flush=True)
    count = (degree + 1) * (degree + 2) * (degree + 3) // 6
    poly = np.random.default_rng(degree).standard_normal(count)
    pts = _points(1000)
    x = torch.from_numpy(pts).cuda()
    S = _net(fallback, sigma=1e-6, poly_degree=degree, poly=poly)
    Z = _net(fallback, sigma=1e-6)
    got = S.predict(x).cpu().numpy() - Z.predict(x).cpu().numpy()
    ref = M.poly_eval(pts, poly, degree, 8.0)
    scale = M.poly_eval(np.abs(pts), np.abs(poly), degree, 8.0)
    assert np.all(np.abs(got - ref) <= 200 * 2.0 ** -53 * (scale + 1.0))
    S.close()
    Z.close()


@pytest.mark.parametrize("n", [1, 31, 32, 33, 127, 128, 129, 161, 1000, 8193, 40001])
def test_gradient_does_not_depend_on_the_row_order(fallback, n):
    """Loss from the predictions, and the gradient under a permutation that
    moves rows into and out of the last tile and partial.  The targets lie
    one below the values, so the sums do not cancel: n FP32 additions of
    terms rounded alike, below 1e-5 of the gradient."""
    import torch
    print(f"[tiles] gradient {n}", flush=True)
    S = _net(fallback, sigma=1.0)
    pts = _points(n)
    x = torch.from_numpy(pts).cuda()
    y = S.predict(x).cpu().numpy()
    t = (y - 1.0).astype(np.float32)
    loss, g = S.loss_grad(x, torch.from_numpy(t).cuda())
    want = np.mean((y - t.astype(np.float64)) ** 2)
    assert abs(loss - want) <= 1e-6 * want
    assert abs(g[-1] - np.mean(2 * (y - t))) <= 1e-5 * abs(g[-1])
    p = np.random.default_rng(n).permutation(n)
    loss2, g2 = S.loss_grad(torch.from_numpy(pts[p].copy()).cuda(), torch.from_numpy(t[p].copy()).cuda())
    assert abs(loss2 - loss) <= 1e-12 * loss
    assert np.linalg.norm(np.asarray(g2, float) - np.asarray(g, float)) <= 1e-5 * np.linalg.norm(np.asarray(g, float))
    S.close()
