"""Which shape-function kernel takes a large float64 call is decided on the device
by the lists' total of pairs: at the edges of that rule, one kernel and one only
works on the lists, and its values are those of smaller calls."""
import numpy as np
import pytest
import torch
from scipy.spatial import cKDTree

import otm_workloads as W
from tests.gpu_common import make_sim, require_gpu

pytestmark = pytest.mark.gpu

N_MP = 4 * 512 * 64


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.fixture(scope="module")
def nearest():
    """Jittered lattice, MPs in Z-order, their 39 nearest nodes, nearest first."""
    rng = np.random.default_rng(3)
    g = np.arange(24.0)
    x = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    x = x + rng.uniform(-0.1, 0.1, x.shape)
    xp = rng.uniform(3.0, 20.0, (N_MP + 1, 3))
    i = (xp * 4).astype(np.int64)
    xp = xp[np.argsort(W._morton3(i[:, 0], i[:, 1], i[:, 2]))]
    return x, xp, cKDTree(x).query(xp, 39)[1]


# (the pairs of n_mp rows of k and one row longer or shorter by ``more``)
@pytest.mark.parametrize("n_mp", [N_MP - 1, N_MP, N_MP + 1])
@pytest.mark.parametrize("k,more", [(24, 0), (31, -1), (31, 0), (38, 0), (38, 1)])
def test_edges_of_the_row_lengths(nearest, n_mp, k, more):
    from paper_2206_08772_amd.sim import lme_shape, read_diag
    x, xp, near = nearest
    xp, near = xp[:n_mp].copy(), near[:n_mp]
    xp[[7, n_mp - 3]] = 40.0                          # outside the hull: not solvable
    K = np.full(n_mp, k)
    K[n_mp // 3] += more
    use = np.arange(near.shape[1]) < K[:, None]
    ids = np.sort(np.where(use, near, x.shape[0]), 1)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    idx = dev(ids[ids < x.shape[0]].astype(np.int32))
    offsets = dev(np.concatenate([[0], np.cumsum(K)]))
    xd, pd = dev(x.T), dev(xp.T)
    lam, N, dN, diag = lme_shape(xd, pd, offsets, idx, 4.0, 1e-13)
    _, d = read_diag(diag)
    assert (d.n_lme_noconv, d.first_lme_noconv) == (2, 7)
    solved = torch.ones(n_mp, dtype=torch.bool, device="cuda")
    solved[[7, n_mp - 3]] = False
    rows = dev(K)
    h = n_mp // 2 + 3
    for a, b in ((0, h), (h, n_mp)):
        q0, q1 = int(offsets[a]), int(offsets[b])
        l2, N2, dN2, _ = lme_shape(xd, pd[:, a:b].contiguous(), (offsets[a:b + 1] - q0).contiguous(),
                                   idx[q0:q1].contiguous(), 4.0, 1e-13)
        g = solved[a:b].repeat_interleave(rows[a:b])
        # |r| <= 1e-13 on both sides moves N by |J^-1 d| |r| N: J > 0.02 inside a
        # lattice at this prior, |d| < 3
        assert float((N[q0:q1] - N2)[g].abs().max()) < 4e-11
        assert float((dN[:, q0:q1] - dN2)[:, g].abs().max()) < 4e-9
        assert float((lam[:, a:b] - l2)[:, solved[a:b]].abs().max()) < 1e-11


@pytest.mark.parametrize("per_radius,skin_h", [(10.6, 0.0), (10.6, 0.12), (13.2, 0.0), (13.2, 0.25)])
@pytest.mark.parametrize("over", [{}, {"kappa": 400.0}, {"scatter": "segmented"}, {"eps_stab": 1.0}])
def test_bodies_are_assembled_once(per_radius, skin_h, over):
    """Bodies of 0.15M (few rows past 27 pairs, or many) and 0.28M MPs: sum N = 1,
    and the nodal masses and forces are the sums of the pairs'."""
    over = dict(over)
    w = W.taylor_rod(h=3.2e-3 / per_radius, seed=2, length=22.4e-3, skin_h=skin_h)
    assert w.n_mp >= (N_MP if per_radius < 11 else 2 * N_MP)
    if "eps_stab" in over:
        over["eps_stab"] = 26.9e9 * w.h ** 2
    sim, p = make_sim(w, **over)
    sim.init()
    sim.run(2)
    sim.check_diag()
    off = sim.offsets
    P = int(off[-1])
    mp = torch.arange(w.n_mp, device="cuda").repeat_interleave(torch.diff(off))
    I = sim.idx[:P].long()
    N = sim.N[:P]
    total = torch.zeros(w.n_mp, dtype=torch.float64, device="cuda").index_add_(0, mp, N)
    assert float((total - 1.0).abs().max()) < 1e-12

    def check(got, pair):
        want = torch.zeros_like(got).index_add_(0, I, pair)
        size = torch.zeros_like(got).index_add_(0, I, pair.abs())
        # up to ~200 terms in another order
        assert float(((got - want).abs() - 1e-13 * size).max()) <= 0.0

    check(sim.m, N * sim.mass[mp])
    if "eps_stab" not in over:
        g, s = sim.dN[:, :P], sim.sigma[:, mp]
        check(sim.f[0], -sim.vol[mp] * (s[0] * g[0] + s[3] * g[1] + s[5] * g[2]))
