"""The real-space term does not depend on the unit of length: every length
times 2^k and beta over 2^k is the same system, with energies over 2^k and
forces over 2^2k (powers of two, so that only the order of additions may
differ), and a box may be any number of times larger than the cutoff."""
import math

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2009_12617_amd as pkg
    return pkg


def dev(a, dtype=np.float64):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).to("cuda")


# (four, two and one wavefront a group of home atoms)
@pytest.mark.parametrize("n", [600, 6000, 17000])
@pytest.mark.parametrize("k", [-200, -100, -40, 40, 70, 200])
def test_units(P, n, k):
    rng = np.random.default_rng(n)
    edges = np.array([1.0, 1.1, 0.95]) * 2.2 * n ** (1.0 / 3.0)
    rcut, beta = min(8.0, 0.94 * edges.min() / 3), 0.36
    pos, q = rng.random((n, 3)) * edges, rng.uniform(-1.0, 1.0, size=n)
    s = 2.0 ** k
    real = P.RealSpace(n)
    f, e = real(dev(pos), dev(q), np.diag(edges), beta, rcut)
    g, h = real(dev(pos * s), dev(q), np.diag(edges * s), beta / s, rcut * s)
    f, g = f.cpu().numpy(), g.cpu().numpy() * s * s
    assert np.linalg.norm(g - f) <= 1e-12 * np.linalg.norm(f)
    assert float(h[0]) * s == pytest.approx(float(e[0]), rel=1e-12)
    assert float(h[1]) * s == pytest.approx(float(e[1]), rel=1e-12)


@pytest.mark.parametrize("edge", [1e3, 1e5, 1e6])
def test_cluster_in_a_large_box(P, edge):
    rng = np.random.default_rng(5)
    n, rcut, beta = 400, 6.0, 0.4
    pos, q = rng.random((n, 3)) * 18.0, rng.uniform(-1.0, 1.0, size=n)
    f, e = P.RealSpace(n)(dev(pos), dev(q), np.diag([edge] * 3), beta, rcut)
    ref = oracle.ewald_real(pos, q, np.diag([edge] * 3), beta, nimg=1, rcut=rcut)
    err = np.linalg.norm(f.cpu().numpy() - ref["forces"])
    assert err <= 1e-11 * np.linalg.norm(ref["forces"])
    assert float(e[0]) == pytest.approx(ref["E_real"], rel=1e-12)


@pytest.mark.parametrize("rcut", [1e-4, 1e-6, 1e-9, 1e-12])
def test_cutoff_far_below_the_box(P, rcut):
    # L / rcut past 2^21 (the product of three such counts is past 64 bits)
    # and past 2^31: the grid has max_cells at most
    rng = np.random.default_rng(6)
    n, beta = 300, 3.0 / rcut
    pos, q = rng.random((n, 3)) * 100.0, rng.uniform(-1.0, 1.0, size=n)
    pos[:40] = rcut * rng.random((40, 3)) * 2.0  # near the origin, where such distances exist
    real = P.RealSpace(n, max_cells=1000)
    f, e = real(dev(pos), dev(q), np.diag([100.0] * 3), beta, rcut)
    f, want, E = f.cpu().numpy(), np.zeros((n, 3)), 0.0
    for i in range(40):
        for j in range(40):
            d = pos[i] - pos[j]
            r = math.sqrt(float(d @ d / rcut / rcut)) * rcut
            if i != j and r <= rcut:
                u = q[i] * q[j] * math.erfc(beta * r) / r
                g = q[i] * q[j] * 2 * beta / math.sqrt(math.pi) * math.exp(-(beta * r) ** 2)
                E += 0.5 * u
                want[i] += (u + g) / r * (d / r)
    f, want = f * rcut * rcut, want * rcut * rcut
    assert np.linalg.norm(f - want) <= 1e-11 * np.linalg.norm(want)
    assert float(e[0]) == pytest.approx(E, rel=1e-11)
