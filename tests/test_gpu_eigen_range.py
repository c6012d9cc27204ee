"""The material-point pass's eigen-decomposition at strains whose squares leave the
range of float64: the Hencky stress of an elastic step against numpy's."""
import numpy as np
import pytest
import torch

import otm_workloads as W
from tests.gpu_common import make_sim, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [1e100, 1e139, 1e141, 1e155, 1e200, 1e250])
def test_hencky_stress_of_huge_strains(size):
    require_gpu()
    w = W.config_by_name("small_rod")
    sim, p = make_sim(w, model=W.MODEL_J2_LINEAR, Y0=1e30, H=0.0)
    sim.init()
    rng = np.random.default_rng(11)
    q, _ = np.linalg.qr(rng.standard_normal((w.n_mp, 3, 3)))
    d0 = rng.uniform(0.2, 1.0, (w.n_mp, 3))
    b = q @ (d0[:, :, None] * np.swapaxes(q, 1, 2))
    b = 0.5 * (b + np.swapaxes(b, 1, 2))
    comp = np.stack([b[:, 0, 0], b[:, 1, 1], b[:, 2, 2], b[:, 0, 1], b[:, 1, 2], b[:, 0, 2]])
    sim.bed.copy_(torch.from_numpy(size * comp))
    sim.Fd.zero_()
    sim.du.zero_()
    sim.f.zero_()
    sim.step()
    d, v = np.linalg.eigh(b)
    e = 0.5 * (np.log(d) + np.log(size))          # log1p(size d): the 1 is far below an ulp
    mu = p["E"] / (2 * (1 + p["nu"]))
    lam = p["E"] * p["nu"] / ((1 + p["nu"]) * (1 - 2 * p["nu"]))
    tau = lam * e.sum(1, keepdims=True) + 2 * mu * e
    want = v @ (tau[:, :, None] * np.swapaxes(v, 1, 2))
    ref = np.stack([want[:, 0, 0], want[:, 1, 1], want[:, 2, 2], want[:, 0, 1], want[:, 1, 2],
                    want[:, 0, 2]])
    got = sim.sigma.cpu().numpy()
    # the eigenvalues' roundings (a few dozen of 1.1e-16 of the largest, five times
    # the smallest) reach the strains, and the strains' own the stress
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= 1e-13 * (3 * lam + 2 * mu) * np.abs(e).max()
