"""The sticky flags of the one-launch step: none on a good step, the non-finite
report of a position and of a charge with the other atoms' forces untouched,
and the fixed-point headroom, each as the separate launches have it."""
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


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda")


def both(plan, pos, q, box):
    """(forces, flags) of the one launch and of the separate ones."""
    f, _ = plan.step(dev(pos), dev(q), box)
    flags = plan.check()
    plan.spread(dev(pos), dev(q), box)
    plan.solve()
    f2 = plan.gather()
    return f.cpu().numpy(), flags, f2.cpu().numpy(), plan.check()


BOX = np.diag([12.4, 12.0, 13.0])


@pytest.mark.parametrize("precision", ["fp32_fixed", "fp32_fixed_half", "fp32_fixed_bf16", "fp64"])
@pytest.mark.parametrize("n", [1, 192, 500])
def test_flags(P, precision, n):
    rng = np.random.default_rng(n)
    pos, q = rng.random((n, 3)) @ BOX, rng.standard_normal(n)
    plan = P.Plan(16, 4, 0.34, max_atoms=n, precision=precision)
    f, flags, f2, flags2 = both(plan, pos, q, BOX)
    assert flags == 0 and flags2 == 0
    bad = n // 2
    others = np.arange(n) != bad
    for value in (np.nan, np.inf, -np.inf):
        p, c = pos.copy(), q.copy()
        p[bad, 1] = value
        c[bad] = value
        for args in ((p, q), (pos, c)):
            f, flags, f2, flags2 = both(plan, *args, BOX)
            assert flags == 1 and flags2 == 1  # PME_FLAG_NONFINITE
            assert np.all(np.isfinite(f[others]))
            if precision == "fp64":  # the order of the grid's additions varies
                assert np.allclose(f[others], f2[others], rtol=1e-11, atol=1e-12)
            else:
                assert np.array_equal(f[others], f2[others])
    assert plan.check() == 0  # cleared


def test_headroom(P):
    # sum |q| 2^F against 2^51, F = 40: 2048 raises the flag, just below does not
    n = 256
    pos = np.random.default_rng(7).random((n, 3)) @ BOX
    plan = P.Plan(16, 4, 0.34, max_atoms=n, frac_bits=40)
    for q, want in ((8.0, 2), (np.nextafter(8.0, 0.0), 0)):
        _, flags, _, flags2 = both(plan, pos, np.full(n, q), BOX)
        assert flags == want and flags2 == want
