"""Calls through a multipole tree of more points than one launch takes (2^25
values, 2^23 fields): the pieces join, and sizes whose launch would pass 2^32
threads (2^30 points) are evaluated."""
import numpy as np
import pytest

from paper_1011_4687_amd import synth

pytestmark = pytest.mark.gpu


def _free():
    import torch
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def _points(n, seed):
    """n points of the 8-bohr cube on the device, in pieces."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.empty((n, 3), dtype=torch.float64, device="cuda")
    for a in range(0, n, 1 << 26):
        x[a:a + (1 << 26)].uniform_(-4.5, 4.5, generator=g)
    return x


def _probe(n, cut):
    """Points on either side of every cut, the first and the last."""
    i = np.unique(np.concatenate([np.arange(0, n, cut), np.arange(0, n, cut) - 1, [n - 1], [n // 3]]))
    return i[(i >= 0) & (i < n)]


@pytest.mark.parametrize("kind,n", [("eval", (1 << 25) + 1001), ("field", (1 << 23) + 1001), ("field", (1 << 30) + 64),
                                    ("cells", (1 << 25) + 129)])
def test_pieces(kind, n):
    """The probed points alone go another way (another order and split): FP32C
    to 1e-6 Ha, fields and cells likewise relative to the largest value."""
    import torch
    from paper_1011_4687_amd.envpot import CellEnvironment, Environment
    if _free() < 60 * n + (8 << 30):
        pytest.skip("needs the memory of the points and values")
    print(f"[pieces] {kind} {n}", flush=True)
    if kind == "cells":
        env, _ = synth.cell_workload(seed=5, n_points=10, n_atoms=4, h=0.3)
        E = CellEnvironment.from_synth(env, precision="fp32c")
        call, cut = E.eval, 1 << 25
    else:
        E = Environment.from_synth(synth.make_fragmented(10, 31), precision="fp32c", neutralize=True)
        call, cut = (E.eval, 1 << 25) if kind == "eval" else (E.eval_field, 1 << 23)
    x = _points(n, 7)
    out = call(x)
    i = torch.from_numpy(_probe(n, cut)).cuda()
    a, b = out[i].cpu().numpy(), call(x[i].contiguous()).cpu().numpy()
    assert np.all(np.isfinite(a))
    assert np.max(np.abs(a - b)) <= 1e-6 * max(1.0, np.abs(b).max())
    del x, out
    E.close()
    torch.cuda.empty_cache()
