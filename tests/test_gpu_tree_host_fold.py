"""A handle whose density is folded on the host (a shell has more primitives
than the update tables index, here without density of its own) and that has a
multipole tree: the tree's records and moments are formed at create.  (Half a
minute: the host normalises the shell over all pairs of its primitives.)"""
import numpy as np
import pytest

from paper_1011_4687_amd import synth

pytestmark = pytest.mark.gpu


def test_tree_after_a_host_fold():
    """Against a handle without the shell, folded on the device, in FP64: 1e-11
    of the largest value, as the tree against every pair."""
    import torch
    from paper_1011_4687_amd.envpot import Environment
    env = synth.make_fragmented(20, 35)
    rp, col, val = env.density_csr()
    shells = [(s.atom, s.l, s.exponents, s.coefs) for s in env.shells]
    n = 32768
    more = shells + [(0, 0, np.geomspace(0.1, 1e4, n), np.ones(n))]
    print("[tree] host fold", flush=True)
    A = Environment(env.xyz, env.Z, env.fragment, more, (np.append(rp, rp[-1]), col, val), precision="fp64")
    B = Environment(env.xyz, env.Z, env.fragment, shells, (rp, col, val), precision="fp64")
    a, b = A.info(), B.info()
    assert a["pairs_built_on_device"] == 0 and b["pairs_built_on_device"] == 1
    assert a["n_pairs"] == b["n_pairs"] >= 8192
    x = torch.from_numpy(synth.points_in_ball(np.random.default_rng(6), 3000, 8.0)).cuda()
    va, vb = A.eval(x).cpu().numpy(), B.eval(x).cpu().numpy()
    assert np.abs(va - vb).max() <= 1e-11 * max(1.0, np.abs(vb).max())
    fa, fb = A.eval_field(x).cpu().numpy(), B.eval_field(x).cpu().numpy()
    assert np.abs(fa - fb).max() <= 1e-11 * max(1.0, np.abs(fb).max())
    A.close()
    B.close()
