"""The assembly of the stabilised residual against sums formed from the step's
own N, grad N and positions: bodies whose workgroups take their fewest MPs,
a few rounds and their most, a partial last round, rows past 16, 32 and 48."""
import pytest
import torch

import otm_workloads as W
from tests.gpu_common import make_sim, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("precision", ["fp64", "mixed", "mixed_storage"])
@pytest.mark.parametrize("per_radius,length,skin_h", [(3.2, 9.6e-3, 0.0), (5.8, 22.4e-3, 0.35),
                                                      (7.9, 30e-3, 0.0), (17.0, 26e-3, 0.0)])
def test_sums_of_its_pairs(precision, per_radius, length, skin_h):
    w = W.taylor_rod(h=3.2e-3 / per_radius, seed=2, length=length, skin_h=skin_h)
    eps = w.material.E / (2 * (1 + w.material.nu)) * w.h ** 2
    sim, p = make_sim(w, precision=precision, eps_stab=eps)
    sim.init()
    sim.run(2)
    sim.check_diag()
    off = sim.offsets
    P = int(off[-1])
    rows = torch.diff(off)
    assert skin_h == 0.0 or int(rows.max()) > 48
    mp = torch.arange(w.n_mp, device="cuda").repeat_interleave(rows)
    I = sim.idx[:P].long()
    N, g, s = sim.N[:P], sim.dN[:, :P].double(), sim.sigma.double()[:, mp]
    v = sim.vol[mp]
    x, xq = sim.xp[:, mp], sim.xp_prev[:, mp]
    xi = sim.x[:, I]
    d, dp = xi - x, (xi - sim.du[:, I]) - xq
    wt = -eps * N / dp.norm(dim=0)
    H = sim.dFm1[:, mp]

    def check(got, terms):
        want, size = torch.zeros_like(got), torch.zeros_like(got)
        for t in terms:
            want.index_add_(0, I, t)
            size.index_add_(0, I, t.abs())
        # ~200 pairs in another order, with 1e-15 of each term
        assert float(((got - want).abs() - 1e-13 * size).max()) <= 0.0

    check(sim.m, [N * sim.mass[mp]])
    sig = ((0, 3, 5), (3, 1, 4), (5, 4, 2))
    # (OTM_MIXED forms the stress part in float32: five roundings of 6e-8)
    for i in range(3):
        part = [-v * s[sig[i][k]] * g[k] for k in range(3)]
        rel = H[3 * i] * dp[0] + H[3 * i + 1] * dp[1] + H[3 * i + 2] * dp[2]
        terms = part + [wt * d[i], -wt * dp[i], -wt * rel]
        if precision != "mixed":
            check(sim.f[i], terms)
            continue
        want, size = torch.zeros_like(sim.m), torch.zeros_like(sim.m)
        for t in terms:
            want.index_add_(0, I, t)
        scale = sum(t.abs() for t in part)
        size.index_add_(0, I, scale * 5e-7 + 1e-13 * (wt * d[i]).abs())
        assert float(((sim.f[i] - want).abs() - size).max()) <= 0.0
