"""The real-space term of boxes that are not evenly filled: forces against the
CPU oracle with dense and empty rows of cells at the sizes where the list of
home groups is made in another way (one-workgroup sort, scan in the fill, scan
of its own, more units than the listing workgroup has threads), and the time
of a slab, which must not depend on the axis it lies across."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
FORCE_RMS = 1e-11


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2009_12617_amd as pkg
    return pkg


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda")


# atoms, box edges, the filled part (low and high corner, in box units), rcut
CASES = [
    (900, (33.0, 33.0, 33.0), ((0, 0, 0.4), (1, 1, 0.6)), 8.0),          # 4 rows of cells in 16
    (4000, (40.0, 40.0, 80.0), ((0, 0, 0.45), (1, 1, 0.7)), 8.0),
    (6000, (40.0, 40.0, 80.0), ((0.3, 0.3, 0.4), (0.7, 0.7, 0.6)), 8.0),
    (9000, (64.0, 64.0, 64.0), ((0, 0, 0), (0.3, 0.3, 0.3)), 8.0),       # scan in the fill
    (3000, (24.0, 144.0, 144.0), ((0, 0, 0.4), (1, 1, 0.6)), 7.9),       # 972 units of one cell
    (20000, (100.0, 100.0, 100.0), ((0.1, 0.4, 0.4), (0.9, 0.8, 0.6)), 8.0),  # a scan of its own
    (6000, (24.0, 320.0, 320.0), ((0, 0.2, 0.2), (1, 0.3, 0.9)), 7.9),   # 4,800 units of one cell
]


@pytest.mark.parametrize("n,edges,part,rcut", CASES)
def test_forces(P, n, edges, part, rcut):
    rng = np.random.default_rng(n)
    lo, hi = np.array(part[0], dtype=float), np.array(part[1], dtype=float)
    pos = (lo + rng.random((n, 3)) * (hi - lo)) * np.array(edges)
    pos[: n // 50] = rng.random((n // 50, 3)) * np.array(edges)  # a few anywhere
    pos = pos[rng.permutation(n)]
    q, box = rng.uniform(-1.0, 1.0, size=n), np.diag(np.array(edges, dtype=float))
    f, e = P.RealSpace(n)(dev(pos), dev(q), box, 0.36, rcut)
    f = f.cpu().numpy()
    if n <= 4000:
        ref = oracle.ewald_real(pos, q, box, 0.36, nimg=1, rcut=rcut)
        want, atoms = ref["forces"], np.arange(n)
        assert float(e[0]) == pytest.approx(ref["E_real"], rel=1e-12)
    else:
        atoms = np.sort(rng.choice(n, size=48, replace=False)).astype(np.int32)
        out = oracle.ewald_real_atoms(pos, q, box, 0.36, atoms, nimg=1, rcut=rcut)
        want = out["forces"] if isinstance(out, dict) else out
    err = np.linalg.norm(f[atoms] - want)
    print(f"force error {err:.2e} of {np.linalg.norm(want):.2e}", flush=True)
    assert err <= FORCE_RMS * np.linalg.norm(want)


def test_slab_time_does_not_depend_on_its_axis(P):
    # 65,535 charges at liquid density in a tenth of the box: across x every
    # row of cells holds the same, across z a tenth of the rows hold all
    rng = np.random.default_rng(1)
    n, edge = 65535, 86.8
    base, q = rng.random((n, 3)) * edge, dev(rng.uniform(-1.0, 1.0, size=n))
    real = P.RealSpace(n)
    f = torch.empty((n, 3), dtype=torch.float64, device="cuda")
    us = {}
    for axis in (0, 2):
        edges = np.full(3, edge)
        edges[axis] *= 10.0
        pos = base.copy()
        pos[:, axis] += 4.0 * edge
        pos = dev(pos)
        best = float("inf")
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                real(pos, q, np.diag(edges), 0.34, 9.0, forces=f)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 1e2)
        us[axis] = best
    print(f"slab across x {us[0]:.1f} us, across z {us[2]:.1f} us", flush=True)
    assert us[2] <= 1.5 * us[0]
