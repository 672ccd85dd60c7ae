"""GPU real-space term at the sizes where its sorting and pair kernels change
course: group and tile remainders, the one-workgroup sort and its limits, the
wavefronts sharing a group, rows of three and of more than 64 cells, sparse
rows (groups cut at cells), and more candidates than one list holds.  Forces
against the CPU oracle (of sampled atoms in the larger systems), at the
tolerances of the existing real-space tests."""
import numpy as np
import pytest
import torch

import oracle
from paper_2009_12617_amd import inputs as I

pytestmark = pytest.mark.gpu
FORCE_RMS = 1e-11


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2009_12617_amd as P
    from paper_2009_12617_amd import _lib
    _lib.load()
    return P


def dev(a, dtype=np.float64):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).to("cuda")


def charges(rng, n, edges):
    pos = rng.uniform(0.0, 1.0, size=(n, 3)) * np.array(edges)
    q = rng.uniform(-1.0, 1.0, size=n)
    return pos, q, np.diag(np.array(edges, dtype=np.float64))


# atoms, box edges, beta, rcut
CASES = [
    (1, (24.0, 24.0, 24.0), 0.35, 7.9),
    (2, (24.0, 24.0, 24.0), 0.35, 7.9),
    (17, (24.0, 24.0, 24.0), 0.35, 7.9),
    (65, (24.0, 40.0, 33.0), 0.35, 7.5),       # 3 x 5 x 4 cells
    (60, (32.0, 32.0, 32.0), 0.35, 7.9),       # 4 cells a row, groups cut at cells
    (1500, (40.0, 24.0, 24.0), 0.35, 7.9),     # 5 x 3 x 3 cells
    (2500, (600.0, 24.0, 24.0), 0.35, 7.9),    # 75 cells a row
    (5121, (50.0, 50.0, 50.0), 0.44, 8.1),     # two wavefronts a group; 32 terms
    (8192, (58.0, 58.0, 58.0), 0.36, 8.0),     # the largest one-workgroup sort
    (8193, (58.0, 58.0, 58.0), 0.36, 8.0),
    (8000, (90.0, 90.0, 90.0), 0.36, 8.0),     # more sub-cells than it takes
    (20000, (90.0, 90.0, 90.0), 0.36, 8.0),    # more sub-cells than a fill scans
]


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("n,edges,beta,rcut", CASES)
def test_shapes(P, n, edges, beta, rcut, accumulate):
    rng = np.random.default_rng(n)
    pos, q, box = charges(rng, n, edges)
    old = rng.normal(size=(n, 3)) if accumulate else np.zeros((n, 3))
    print(f"real space n={n} edges={edges} rcut={rcut} accumulate={accumulate}", flush=True)
    f = dev(old)
    _, e = P.RealSpace(n)(dev(pos), dev(q), box, beta, rcut, forces=f, accumulate=accumulate)
    f = f.cpu().numpy() - old
    if n <= 2500:
        ref = oracle.ewald_real(pos, q, box, beta, nimg=1, rcut=rcut)
        want, atoms = ref["forces"], np.arange(n)
        assert float(e[0]) == pytest.approx(ref["E_real"], rel=1e-12, abs=1e-13)
        assert float(e[1]) == pytest.approx(ref["E_self"], rel=1e-13)
    else:
        atoms = np.sort(rng.choice(n, size=48, replace=False)).astype(np.int32)
        out = oracle.ewald_real_atoms(pos, q, box, beta, atoms, nimg=1, rcut=rcut)
        want = out["forces"] if isinstance(out, dict) else out
    err = np.linalg.norm(f[atoms] - want)
    print(f"force error {err:.2e} of {np.linalg.norm(want):.2e}", flush=True)
    assert err <= FORCE_RMS * np.linalg.norm(want)


def test_dense_cluster(P):
    # 3,000 charges in a 9 A cube: every one a candidate of every group, more
    # than one list of 2,048 holds
    rng = np.random.default_rng(71)
    n = 3000
    pos = 10.0 + rng.uniform(0.0, 9.0, size=(n, 3))
    q = rng.uniform(-1.0, 1.0, size=n)
    box = np.diag([27.0] * 3)
    f, e = P.RealSpace(n)(dev(pos), dev(q), box, 0.35, 8.9)
    ref = oracle.ewald_real(pos, q, box, 0.35, nimg=1, rcut=8.9)
    err = np.linalg.norm(f.cpu().numpy() - ref["forces"])
    print(f"force error {err:.2e} of {np.linalg.norm(ref['forces']):.2e}", flush=True)
    assert err <= FORCE_RMS * np.linalg.norm(ref["forces"])
    assert float(e[0]) == pytest.approx(ref["E_real"], rel=1e-12)


@pytest.mark.parametrize("n", [500, 9000])
def test_nonfinite_atom_leaves_the_others(P, n):
    # an atom at a NaN position has no pairs: the others' forces are those
    # without it, its own is zero
    rng = np.random.default_rng(72)
    pos, q, box = charges(rng, n, (50.0, 50.0, 50.0))
    bad = n // 3
    keep = np.arange(n) != bad
    want, ew = P.RealSpace(n)(dev(pos[keep]), dev(q[keep]), box, 0.36, 8.0)
    pos[bad, 1] = np.nan
    got, eg = P.RealSpace(n)(dev(pos), dev(q), box, 0.36, 8.0)
    got, want = got.cpu().numpy(), want.cpu().numpy()
    assert np.all(got[bad] == 0.0)
    assert np.linalg.norm(got[keep] - want) <= FORCE_RMS * np.linalg.norm(want)
    assert float(eg[0]) == pytest.approx(float(ew[0]), rel=1e-12)
