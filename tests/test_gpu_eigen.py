"""The material-point pass's eigen-decomposition: an unloaded step on elastic
strains with equal, nearly equal, widely spread and vanishing eigenvalues or
off-diagonals, against the Hencky stress of numpy's decomposition."""
import numpy as np
import pytest
import torch

import otm_workloads as W
from tests.gpu_common import make_sim, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def strains(n, size):
    """n symmetric matrices of the given size: rotated diagonals of every kind,
    some with off-diagonals scaled down, some diagonal, some zero."""
    rng = np.random.default_rng(7)
    q, _ = np.linalg.qr(rng.standard_normal((n, 3, 3)))
    d = rng.uniform(-1, 1, (n, 3))
    kind = np.arange(n) % 8
    d[kind == 1, 1] = d[kind == 1, 0]
    d[kind == 2] = d[kind == 2][:, :1]
    d[kind == 3, 1] = d[kind == 3, 0] * (1 + 1e-13)
    d[kind == 4] *= np.array([1, 1e-6, 1e-12])
    b = q @ (d[:, :, None] * np.swapaxes(q, 1, 2))
    b = 0.5 * (b + np.swapaxes(b, 1, 2))
    off = 1 - np.eye(3)
    b[kind == 5] *= np.eye(3) + 1e-9 * off
    b[kind == 6] *= np.eye(3) + 1e-170 * off
    b[kind == 7] = 0.0
    b[8] = np.diag([1.0, 1.0, -1.0])
    b[9] = np.array([[0, -1, 0], [-1, 0, 0], [0, 0, 0.5]])
    return size * b


# a few dozen roundings of 1.1e-16 of the largest entry; OTM_MIXED_STORAGE rounds
# sigma to float32 once (6e-8 of it)
@pytest.mark.parametrize("precision,tol", [("fp64", 4e-14), ("mixed_storage", 1e-7)])
@pytest.mark.parametrize("size", [1e-3, 1e-9, 1e-30])
def test_hencky_stress(precision, tol, size):
    w = W.config_by_name("small_rod")
    sim, p = make_sim(w, precision=precision)
    sim.init()
    b = strains(w.n_mp, size)
    dt = sim.bed.dtype
    comp = np.stack([b[:, 0, 0], b[:, 1, 1], b[:, 2, 2], b[:, 0, 1], b[:, 1, 2], b[:, 0, 2]])
    sim.bed.copy_(torch.from_numpy(comp).to(dt))
    stored = sim.bed.double().cpu().numpy()
    sim.Fd.zero_()
    sim.du.zero_()
    sim.f.zero_()
    sim.step()
    s = stored
    b = np.stack([np.stack([s[0], s[3], s[5]]), np.stack([s[3], s[1], s[4]]),
                  np.stack([s[5], s[4], s[2]])]).transpose(2, 0, 1)
    d, v = np.linalg.eigh(b)
    e = 0.5 * np.log1p(d)
    mu = p["E"] / (2 * (1 + p["nu"]))
    lam = p["E"] * p["nu"] / ((1 + p["nu"]) * (1 - 2 * p["nu"]))
    tau = lam * e.sum(1, keepdims=True) + 2 * mu * e
    want = v @ (tau[:, :, None] * np.swapaxes(v, 1, 2))
    got = sim.sigma.double().cpu().numpy()
    ref = np.stack([want[:, 0, 0], want[:, 1, 1], want[:, 2, 2], want[:, 0, 1], want[:, 1, 2],
                    want[:, 0, 2]])
    elastic = sim.epsbar.cpu().numpy() == 0.0
    assert elastic.sum() > 0.5 * w.n_mp
    scale = (3 * lam + 2 * mu) * np.abs(b).max((1, 2))
    assert np.isfinite(got).all()
    assert (np.abs(got - ref)[:, elastic] <= tol * scale[elastic]).all()
