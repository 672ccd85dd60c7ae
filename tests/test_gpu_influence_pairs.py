"""Influence function taken for mirrored modes together (orthorhombic cells) and
for m and -m together with the Nyquist modes apart (general cells): the energy,
the virial and the convolved spectrum, against the plain formula on every mode
in FP64 -- each index averaged over its two signs at the Nyquist point.  Grids
whose halves do and do not fill whole wavefronts, both kinds of cell; FP64
plans, where nothing but rounding (some hundred FP64 operations per mode)
separates the two: 1e-12.  The other convolutions in FP32, 2e-6."""
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
@pytest.mark.parametrize("K,conv", [(16, 0), (24, 0), (36, 0), (48, 0), (72, 0), ((48, 32, 64), 0),
                                    (96, 0), ((32, 32, 64), 1), (96, 1), (32, 2), (64, 2)], ids=str)
def test_energy_virial_and_potential(P, K, conv, general):
    shape = (K,) * 3 if np.ndim(K) == 0 else K
    # (the split convolution holds part of the factors in LDS: enough atoms
    # that the spreading before it leaves negative integers, NaN as FP64, there)
    prec = "fp64" if conv == 0 else "fp32_fixed"
    pos, q, _ = I.water_box(60 if conv == 0 else 6000, 0.8 * shape[0], 11)
    edges = 0.8 * np.asarray(shape, dtype=np.float64)
    box = np.diag(edges)
    if general:
        box[1, 0], box[2, 0], box[2, 1] = 0.13 * edges[0], -0.08 * edges[0], 0.11 * edges[1]
    pos = pos / (0.8 * shape[0]) @ box
    plan = P.Plan(shape, 4, 0.34, max_atoms=len(q), precision=prec)
    dp, dq = (torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda") for a in (pos, q))
    plan.set_debug(True)
    plan.set_tuning(conv=conv)
    _, ev = plan.step(dp, dq, box)
    grid = plan.debug_grid(0).cpu().numpy().astype(np.float64)
    want, phi = reference(grid if conv == 0 else grid / 2.0 ** plan.frac_bits, box, 0.34, 4)
    bar = 1e-12 if conv == 0 else 2e-6  # FP32 transforms, as the other parity tests
    got = ev.cpu().numpy()
    assert np.abs(got - want).max() <= bar * np.abs(want).max()
    have = plan.debug_grid(2).cpu().numpy()
    assert np.abs(have - phi).max() <= bar * np.abs(phi).max()
    # the one-launch and the separate steps agree
    plan.set_debug(False)
    _, again = plan.step(dp, dq, box)
    assert np.abs(again.cpu().numpy() - want).max() <= bar * np.abs(want).max()
