"""The multipole tree against evaluation without it (ENVPOT_NO_TREE=1 at
create: every pair, nucleus and cell at every point), over what the tree can
meet: points inside, around and far from the environment, every split
factor, more fragment groups than one pass over the roots takes, one group
of everything, groups without pairs, and density updates.

Tolerances, fixed beforehand from the precisions' own: FP64 values agree to
1e-12 of the sum of the terms' magnitudes (here A >= 10 Ha, taken as 1e-11
Ha and 1e-11 Ha/bohr times the largest field); FP32C potentials to 4e-6 Ha
(both sides are within 2e-6 of the exact value), fields to 4e-6 relative."""
import os

import numpy as np
import pytest

from paper_1011_4687_amd import synth

pytestmark = pytest.mark.gpu

TOL_V = {"fp64": 1e-11, "fp32c": 4e-6}
TOL_E = {"fp64": 1e-11, "fp32c": 4e-6}


def _no_tree(make):
    os.environ["ENVPOT_NO_TREE"] = "1"
    try:
        return make()
    finally:
        os.environ.pop("ENVPOT_NO_TREE")


def _cuda(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _regroup(env, how):
    """(xyz, Z, fragment, shells, P) with the fragment ids changed."""
    frag = env.fragment.copy()
    Z = env.Z.copy()
    xyz = env.xyz.copy()
    if how == "one":
        frag[:] = -1
    elif how == "nuclei":  # two more groups that hold nuclei only
        xyz = np.concatenate([xyz, [[12.0, 3.0, -9.0], [12.5, 3.0, -9.0], [-20.0, 1.0, 2.0]]])
        Z = np.concatenate([Z, [1.0, 2.0, 3.0]])
        frag = np.concatenate([frag, [90, 90, 91]]).astype(np.int32)
    return xyz, Z, frag, [(s.atom, s.l, s.exponents, s.coefs) for s in env.shells], env.density_csr()


def _points(env, where, n, seed=11):
    rng = np.random.default_rng(seed)
    inside = synth.points_in_ball(rng, n, env.r_qm)
    lo, hi = env.xyz.min(0) - 5.0, env.xyz.max(0) + 5.0
    if where == "sphere":
        return inside
    if where == "among":  # among the environment's atoms, some within 0.05 bohr of one
        p = rng.uniform(lo, hi, (n, 3))
        k = n // 8
        p[:k] = env.xyz[rng.integers(0, len(env.xyz), k)] + rng.normal(size=(k, 3)) * 0.05
        return p
    far = inside + np.array([300.0, -250.0, 90.0])
    return np.concatenate([inside[: n // 3], far[: n // 3], rng.uniform(lo, hi, (n - 2 * (n // 3), 3))])


def _close(A, B, x, precision, what):
    va, vb = A.eval(x).cpu().numpy(), B.eval(x).cpu().numpy()
    dv = np.abs(va - vb).max()
    fa, fb = A.eval_field(x).cpu().numpy(), B.eval_field(x).cpu().numpy()
    de = np.abs(fa[:, 1:] - fb[:, 1:]).max() / max(1.0, np.abs(fb[:, 1:]).max())
    df = np.abs(fa[:, 0] - vb).max()
    print(f"[tree] {what} {precision}: max |dV| {dv:.2e}, of the field's V {df:.2e}, |dE| {de:.2e}", flush=True)
    scale = max(1.0, np.abs(vb).max())
    assert dv <= TOL_V[precision] * scale
    assert df <= TOL_V[precision] * scale
    assert de <= TOL_E[precision]


@pytest.mark.parametrize("precision", ["fp64", "fp32c"])
@pytest.mark.parametrize("where", ["sphere", "among", "mixed"])
@pytest.mark.parametrize("groups", ["fragments", "one", "nuclei"])
def test_tree_equals_every_pair(precision, where, groups):
    from paper_1011_4687_amd.envpot import Environment
    env = synth.make_fragmented(120, 31)
    args = _regroup(env, groups)
    A = Environment(*args, precision=precision)
    B = _no_tree(lambda: Environment(*args, precision=precision))
    try:
        assert A.info()["device_bytes"] > B.info()["device_bytes"]  # there is a tree
        for n in (1, 63, 129, 3001):
            _close(A, B, _cuda(_points(env, where, max(n, 8))[:n]), precision, f"{groups} {where} n={n}")
    finally:
        A.close()
        B.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32c"])
def test_every_split_many_groups(precision):
    """3000 atoms: 300 groups (the roots take two passes, a block meets more
    accepted nodes than a wave's list holds), every split factor."""
    from paper_1011_4687_amd.envpot import Environment
    env = synth.make_fragmented(3000, 32)
    A = Environment.from_synth(env, precision=precision, neutralize=True)
    B = _no_tree(lambda: Environment.from_synth(env, precision=precision, neutralize=True))
    try:
        x = _cuda(_points(env, "mixed", 1500))
        vb = B.eval(x).cpu().numpy()
        fb = B.eval_field(x).cpu().numpy()
        for k in range(9):
            os.environ["ENVPOT_SPLIT_LOG2"] = os.environ["ENVPOT_FIELD_SPLIT_LOG2"] = str(k)
            for np_ in (1, 2):
                os.environ["ENVPOT_NP"] = os.environ["ENVPOT_FIELD_NP"] = str(np_)
                va, fa = A.eval(x).cpu().numpy(), A.eval_field(x).cpu().numpy()
                assert np.abs(va - vb).max() <= TOL_V[precision] * max(1.0, np.abs(vb).max()), (k, np_)
                assert np.abs(fa - fb).max() <= TOL_E[precision] * max(1.0, np.abs(fb).max()), (k, np_)
                assert np.array_equal(va, A.eval(x).cpu().numpy()), (k, np_)
    finally:
        for e in ("ENVPOT_SPLIT_LOG2", "ENVPOT_FIELD_SPLIT_LOG2", "ENVPOT_NP", "ENVPOT_FIELD_NP"):
            os.environ.pop(e, None)
        A.close()
        B.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32c"])
def test_tree_follows_the_density(precision):
    """After a density update the tree's moments and radii are the new
    density's: equal to a handle built with it; a zero density leaves the
    nuclei."""
    from paper_1011_4687_amd.envpot import Environment
    env = synth.make_fragmented(80, 33)
    rp, col, val = env.density_csr()
    rng = np.random.default_rng(5)
    s = rng.uniform(0.5, 1.5, env.nbf)
    rows = np.repeat(np.arange(env.nbf), np.diff(rp))
    new = (rp, col, val * s[rows] * s[col])
    shells = [(q.atom, q.l, q.exponents, q.coefs) for q in env.shells]
    A = Environment(env.xyz, env.Z, env.fragment, shells, (rp, col, val), precision=precision)
    C = Environment(env.xyz, env.Z, env.fragment, shells, new, precision=precision)
    x = _cuda(_points(env, "mixed", 2000))
    try:
        A.update_density(new)
        va, vc = A.eval(x).cpu().numpy(), C.eval(x).cpu().numpy()
        assert np.abs(va - vc).max() <= 1e-11 * max(1.0, np.abs(vc).max())
        A.update_density((rp, col, np.zeros_like(val)))
        v = A.eval(x).cpu().numpy()
        p = x.cpu().numpy()
        d = np.linalg.norm(p[:, None] - env.xyz[None], axis=2)
        ref = (env.Z[None] / d).sum(axis=1)
        assert np.abs(v - ref).max() <= 1e-12 * np.abs(ref).max()
    finally:
        A.close()
        C.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32c"])
@pytest.mark.parametrize("n", [1, 130, 2048, 40000])
def test_cells_tree_equals_every_cell(precision, n):
    """The cell sum through the tree: FP64 to 1e-13 of the sum of the cells'
    magnitudes, FP32C to 1e-6 Ha (the direct sum's own error)."""
    from paper_1011_4687_amd.envpot import CellEnvironment
    env, pts = synth.cell_workload(seed=77, n_points=n, n_atoms=6, h=0.25)
    A = CellEnvironment.from_synth(env, precision=precision)
    B = _no_tree(lambda: CellEnvironment.from_synth(env, precision=precision))
    try:
        for shift in (0.0, 5.0, 400.0):  # among the cells too
            x = _cuda(pts + shift * np.array([1.0, 0.3, -0.2]) + 1e-3)
            va, vb = A.eval(x).cpu().numpy(), B.eval(x).cpu().numpy()
            tol = 1e-13 * env.Z.sum() * 4 if precision == "fp64" else 1e-6
            assert np.abs(va - vb).max() <= tol * max(1.0, np.abs(vb).max()), shift
    finally:
        A.close()
        B.close()
