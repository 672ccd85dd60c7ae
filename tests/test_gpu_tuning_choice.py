"""What a chosen tuning makes a step run, and what writing a tuning back leaves
alone: the binning chunk of a lone step (read from the per-workgroup charge
sums it leaves in the workspace), the one-launch step of small systems, and
the autotuner on them."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
CHUNKS = (256, 512, 1024)


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2009_12617_amd as pkg
    return pkg


def system(n, edge, seed=3):
    rng = np.random.default_rng(seed)
    pos = torch.from_numpy(rng.random((n, 3)) * edge).to("cuda")
    return pos, np.diag([edge] * 3)


class Chunk:
    """The binning chunk of a plan's step: every charge is c, so a workgroup
    of m atoms leaves the sum m c (exact), and c is another each time."""

    def __init__(self):
        self.k = 0

    def ran(self, plan, n, edge):
        self.k += 1
        c = 1.0 + self.k * 2.0 ** -10
        pos, box = system(n, edge)
        plan.step(pos, torch.full((n,), c, dtype=torch.float64, device="cuda"), box)
        off = -plan._ws.data_ptr() % 256
        ws = plan._ws[off:off + plan.workspace_bytes // 8 * 8].view(torch.float64)
        found = [m for m in CHUNKS if n // m and int((ws == m * c).sum()) == n // m]
        assert len(found) == 1, found
        return found[0]


@pytest.mark.parametrize("n", [4095, 12000, 30000])
def test_writing_a_tuning_back_keeps_the_chunk(P, n):
    edge, chunk = 64.0, Chunk()
    plan = P.Plan(32, 4, 0.35, max_atoms=n)
    default = plan.tuning
    first = chunk.ran(plan, n, edge)
    plan.set_tuning(conv=default["conv"])
    assert chunk.ran(plan, n, edge) == first
    plan.set_tuning(**plan.tuning)
    assert chunk.ran(plan, n, edge) == first
    # a failed autotune restores what it found
    pos, box = system(n + 1, edge)
    q = torch.ones(n + 1, dtype=torch.float64, device="cuda")
    with pytest.raises(RuntimeError):
        plan.autotune(pos, q, box, reps=1)  # one atom too many
    assert plan.tuning == default
    assert chunk.ran(plan, n, edge) == first


@pytest.mark.parametrize("n", [4095, 30000])
def test_smaller_chunks_run_as_set(P, n):
    edge, chunk = 64.0, Chunk()
    plan = P.Plan(32, 4, 0.35, max_atoms=n)
    for m in (512, 256):
        plan.set_tuning(bin_chunk=m)
        assert chunk.ran(plan, n, edge) == m
    plan.set_tuning(bin_chunk=1024)
    assert chunk.ran(plan, n, edge) == chunk.ran(P.Plan(32, 4, 0.35, max_atoms=n), n, edge)


def small(n=192):
    rng = np.random.default_rng(n)
    pos, box = system(n, 12.4, seed=n)
    return pos, torch.from_numpy(rng.standard_normal(n)).to("cuda"), box


@pytest.mark.parametrize("precision", ["fp32_fixed", "fp32_fixed_half"])
@pytest.mark.parametrize("change", [{"interp": 1}, {"bin_chunk": 256}])
def test_small_step_runs_the_variants_set(P, precision, change):
    # the one launch adds its energy in an order of its own; under chosen
    # variants a step has the bits of spread, solve and gather
    pos, q, box = small()
    plan = P.Plan(16, 4, 0.34, max_atoms=192, precision=precision)
    default = plan.tuning
    f1, ev1 = plan.step(pos, q, box)
    plan.set_tuning(**change)
    f, ev = plan.step(pos, q, box)
    plan.spread(pos, q, box)
    ev2 = plan.solve()
    f2 = plan.gather()
    assert torch.equal(ev, ev2) and torch.equal(f, f2)
    assert not torch.equal(ev1, ev2) and torch.equal(f1, f2)
    # the built-in choice back: the one launch again
    plan.set_tuning(**default)
    f, ev = plan.step(pos, q, box)
    assert torch.equal(ev, ev1) and torch.equal(f, f1)


def test_autotune_of_a_small_system_measures_both_forms(P):
    # the chain takes 18 us to the one launch's 13
    pos, q, box = small()
    plan = P.Plan(16, 4, 0.34, max_atoms=192)
    default = plan.tuning
    r = plan.autotune(pos, q, box, reps=50)
    times = {tuple(c.values()): us for c, us in r["candidates"] if us is not None}
    mine = times.pop(tuple(default.values()))
    print(f"built-in {mine:.2f} us, others {min(times.values()):.2f} us and more", flush=True)
    assert min(times.values()) > 1.15 * mine
    assert r["best"] == default and plan.tuning == default
