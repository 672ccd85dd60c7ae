"""The one-launch step of small systems against the separate launches (spread,
solve, gather), which do the same arithmetic: the same forces bit for bit in
the FP32 precisions; in FP64 the order of the grid's additions varies, by a few
units of the last place.  Sizes at the edges of a wavefront, of the thread
groups that share an atom's planes and of the range where the step takes one
launch, and one bucket holding every atom."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2009_12617_amd as pkg
    return pkg


@pytest.mark.parametrize("precision", ["fp32_fixed", "fp32_fixed_half", "fp32_fixed_bf16", "fp64"])
@pytest.mark.parametrize("p", [4, 6])
@pytest.mark.parametrize("n", [1, 64, 65, 193, 256, 257, 320, 576, 577])
def test_one_launch_equals_the_chain(P, precision, p, n):
    rng = np.random.default_rng(n + p)
    plan = P.Plan(16, p, 0.34, max_atoms=n, precision=precision)
    q = torch.from_numpy(rng.standard_normal(n)).to("cuda")
    for box in (np.diag([12.5, 12.0, 13.0]), np.array([[12.5, 0, 0], [1.5, 12.0, 0], [0.7, -1.0, 13.0]])):
        pos = (rng.random((n, 3)) * 3 - 1) @ box
        if n == 320:
            pos = pos[:1] + 0.01 * rng.random((n, 3))
        pos = torch.from_numpy(np.ascontiguousarray(pos)).to("cuda")
        base = torch.ones((n, 3), dtype=torch.float64, device="cuda")
        added, ev = plan.step(pos, q, box, forces=base.clone(), accumulate=True)
        again = plan.gather()  # what the one launch left in the workspace
        plan.spread(pos, q, box)
        ev2 = plan.solve()
        want = plan.gather()
        scale = float(want.abs().max())
        if precision == "fp64":
            assert float((again - want).abs().max()) <= 1e-12 * scale
            assert float((added - (want + base)).abs().max()) <= 1e-12 * max(scale, 1.0)
        else:
            assert torch.equal(again, want)
            assert torch.equal(added, want + base)
        assert float((ev - ev2).abs().max()) <= 1e-12 * float(ev2.abs().max())
        assert plan.flags() == 0 if hasattr(plan, "flags") else True
