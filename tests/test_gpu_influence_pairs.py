"""Influence function taken for mirrored modes together (orthorhombic cells) and
for m and -m together with the Nyquist modes apart (general cells): the energy,
the virial and the convolved spectrum, against the plain formula on every mode
in FP64 -- each index averaged over its two signs at the Nyquist point.  Grids
whose halves do and do not fill whole wavefronts, both kinds of cell; FP64
plans, where nothing but rounding (some hundred FP64 operations per mode)
separates the two: 1e-12."""
import itertools

import numpy as np
import pytest
import torch

from paper_2009_12617_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2009_12617_amd as pkg
    return pkg


def moduli(K, p):
    m4 = lambda n, x: (max(0.0, 1 - abs(x - 1)) if n == 2 else
                       (x * m4(n - 1, x) + (n - x) * m4(n - 1, x - 1)) / (n - 1))
    w = np.array([m4(p, k + 1.0) for k in range(p - 1)])
    b = (w[None] * np.exp(2j * np.pi * np.outer(np.arange(K), np.arange(p - 1)) / K)).sum(1)
    return 1.0 / np.abs(b) ** 2


def reference(grid, box, beta, p):
    K3, K2, K1 = grid.shape
    F = np.fft.fftn(grid)  # [z, y, x]
    rec = np.linalg.inv(box).T  # rows a*_a
    V = abs(np.linalg.det(box))
    B = (moduli(K3, p)[:, None, None] * moduli(K2, p)[None, :, None] * moduli(K1, p)[None, None])
    idx = np.meshgrid(*(np.fft.fftfreq(K, 1.0 / K) for K in (K3, K2, K1)), indexing="ij")
    E, vir, G = 0.0, np.zeros(6), np.zeros(grid.shape)
    for sg in itertools.product((1, -1), repeat=3):
        # a Nyquist index takes each sign in half of the terms, another index its own
        m = [np.where(2 * np.abs(i) == K, s * np.abs(i), i) for i, K, s in zip(idx, (K3, K2, K1), sg)]
        v = [m[2] * rec[0, c] + m[1] * rec[1, c] + m[0] * rec[2, c] for c in range(3)]
        sq = v[0] ** 2 + v[1] ** 2 + v[2] ** 2
        sq[0, 0, 0] = 1.0
        g = B * np.exp(-np.pi ** 2 * sq / beta ** 2) / (np.pi * V * sq) / 8
        g[0, 0, 0] = 0.0
        G += g
        e = 0.5 * g * np.abs(F) ** 2
        E += e.sum()
        u = 1 / sq + np.pi ** 2 / beta ** 2
        for k, (a, b) in enumerate(((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))):
            vir[k] += (e * ((a == b) - 2 * u * v[a] * v[b])).sum()
    return np.concatenate([[E], vir]), np.fft.ifftn(G * F).real * grid.size


@pytest.mark.parametrize("general", [False, True], ids=["orthorhombic", "general"])
@pytest.mark.parametrize("K", [16, 24, 36, 48, 72, (48, 32, 64), 96], ids=str)
def test_energy_virial_and_potential(P, K, general):
    shape = (K,) * 3 if np.ndim(K) == 0 else K
    pos, q, _ = I.water_box(60, 0.8 * shape[0], 11)
    edges = 0.8 * np.asarray(shape, dtype=np.float64)
    box = np.diag(edges)
    if general:
        box[1, 0], box[2, 0], box[2, 1] = 0.13 * edges[0], -0.08 * edges[0], 0.11 * edges[1]
    pos = pos / (0.8 * shape[0]) @ box
    plan = P.Plan(shape, 4, 0.34, max_atoms=len(q), precision="fp64")
    dp, dq = (torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda") for a in (pos, q))
    plan.set_debug(True)
    plan.set_tuning(conv=0)
    _, ev = plan.step(dp, dq, box)
    want, phi = reference(plan.debug_grid(0).cpu().numpy(), box, 0.34, 4)
    got = ev.cpu().numpy()
    assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max()
    have = plan.debug_grid(2).cpu().numpy()
    assert np.abs(have - phi).max() <= 1e-12 * np.abs(phi).max()
    # the one-launch and the separate steps agree
    plan.set_debug(False)
    _, again = plan.step(dp, dq, box)
    assert np.abs(again.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()
