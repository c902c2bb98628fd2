"""Splits of a batch plan whose handles have multipole trees: a plan of few
blocks is not slower than its instances one after the other (each item tests
its trees' nodes again, so too many items cost more than they spread)."""
import numpy as np
import pytest

from paper_1011_4687_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32c", "fp64"])
@pytest.mark.parametrize("count,n", [(8, 2000), (64, 200)])
def test_plan_is_no_slower_than_its_instances(precision, count, n):
    """Instances of 13,000 to 27,000 pairs (8 of 2000 points in FP64: 1220 us as one
    plan with sixteen items per workgroup, 1060 one after the other).  The values
    are those of single calls, to the tolerances of another split."""
    import torch
    from paper_1011_4687_amd.envpot import Batch, Environment
    print(f"[splits] {precision} {count} x {n}", flush=True)
    base = [Environment.from_synth(synth.make_fragmented(10, 31 + i), precision=precision, neutralize=True)
            for i in range(8)]
    hs = [base[i % 8] for i in range(count)]
    xs = [torch.from_numpy(synth.points_in_ball(np.random.default_rng(i), n, 8.0)).cuda() for i in range(count)]
    outs = [torch.empty(n, dtype=torch.float64, device="cuda") for _ in xs]
    one = [torch.empty_like(o) for o in outs]
    B, s = Batch(hs), torch.cuda.Stream()

    def singles():
        for h, x, o in zip(hs, xs, one):
            h.eval(x, out=o, stream=s)

    def least(call):
        t = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            with torch.cuda.stream(s):
                a.record()
                call()
                b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return min(t)

    torch.cuda.synchronize()
    t_plan, t_one = least(lambda: B.eval(xs, outs, stream=s)), least(singles)
    print(f"[splits] plan {1e3 * t_plan:.0f} us, singles {1e3 * t_one:.0f} us", flush=True)
    tol = 1e-6 if precision == "fp32c" else 1e-11
    for o, r in zip(outs, one):
        assert (o - r).abs().max().item() <= tol
    assert t_plan <= 0.8 * t_one
    B.close()
    for h in base:
        h.close()
