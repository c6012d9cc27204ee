"""The pipelined shape-function kernel (131,072 MPs and more, float64) against
the kernel that smaller calls take, over rows of every length (none, one, up to
and past the 40 pairs it keeps in registers), MPs no solve converges for,
capacities of both parities and a partial last round; calls with float32 grad
N, which keep that kernel at every size; and the fused assembly against the
sums formed from its own N and grad N."""
import numpy as np
import pytest
import torch

import otm_workloads as W
from tests.gpu_common import make_sim, require_gpu

pytestmark = pytest.mark.gpu

N_MP = 4 * 512 * 64


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def cloud(n_mp, seed=3):
    """Jittered lattice of spacing 1; MPs inside it in Z-order, a few of them
    outside its hull or out of reach of every node."""
    rng = np.random.default_rng(seed)
    g = np.arange(24.0)
    x = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    x = x + rng.uniform(-0.1, 0.1, x.shape)
    xp = rng.uniform(2.0, 21.0, (n_mp, 3))
    i = (xp * 4).astype(np.int64)
    xp = xp[np.argsort(W._morton3(i[:, 0], i[:, 1], i[:, 2]))]
    xp[5] = xp[70] = xp[n_mp - 2] = (60.0, 60.0, 60.0)        # no node in reach
    xp[6] = xp[1000] = xp[n_mp - 1] = (24.2, 11.0, 11.0)      # outside the hull
    xp[200] = (23.1, 23.1, 23.9)                              # few nodes, outside
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a.T)).cuda()  # noqa: E731
    return dev(x), dev(xp)


@pytest.mark.parametrize("n_mp", [N_MP, N_MP + 37])
@pytest.mark.parametrize("radius,extra", [(1.86, 0), (1.86, 1), (2.05, 1), (2.05, 0), (2.4, 0)])
def test_pipelined_matches_small_calls(n_mp, radius, extra):
    from paper_2206_08772_amd.sim import build_neighbors, lme_shape, read_diag
    x, xp = cloud(n_mp)
    offsets, idx = build_neighbors(x, xp, radius, radius * 1.0001)
    P = idx.numel()
    pad = (P + extra) % 2 + 2                     # capacity P + pad: even, odd with ``extra``
    idx = torch.cat([idx, torch.zeros(pad, dtype=torch.int32, device="cuda")])
    assert (P + pad) % 2 == extra
    lam, N, dN, diag = lme_shape(x, xp, offsets, idx, 4.0, 1e-14)
    _, d = read_diag(diag)
    noconv, first = 0, 2 ** 64 - 1
    rows = torch.diff(offsets)
    assert int(rows.min()) == 0 and int(rows.max()) > (32 if radius < 2 else 40)
    h = n_mp // 2 + 11                            # two calls of the other kernel
    for a, b in ((0, h), (h, n_mp)):
        o = (offsets[a:b + 1] - offsets[a]).contiguous()
        q0, q1 = int(offsets[a]), int(offsets[b])
        l2, N2, dN2, g2 = lme_shape(x, xp[:, a:b].contiguous(), o, idx[q0:q1].contiguous(), 4.0,
                                    1e-14)
        _, d2 = read_diag(g2)
        noconv += d2.n_lme_noconv
        if d2.n_lme_noconv:
            first = min(first, d2.first_lme_noconv + a)
        # rows the other kernel solved: consistency of the shape functions
        pos = xp[:, a:b].repeat_interleave(rows[a:b], dim=1) - x[:, idx[q0:q1].long()]
        res = torch.zeros(3, b - a, dtype=torch.float64, device="cuda")
        mp = torch.arange(b - a, device="cuda").repeat_interleave(rows[a:b])
        res.index_add_(1, mp, pos * N2)
        good = (res.norm(dim=0) <= 1e-12) & (rows[a:b] > 0) & torch.isfinite(l2).all(0)
        assert int((~good).sum()) <= 16
        use = good[mp]
        # |r| <= 1e-14 on both sides moves N by |J^-1 d| |r| N < 1e-12 away from
        # the hull, where J > 0.1; the outermost accepted MPs lie 2 inside it
        assert float((N[q0:q1] - N2)[use].abs().max()) < 1e-11
        assert float((dN[:, q0:q1] - dN2)[:, use].abs().max()) < 1e-11
        assert float((lam[:, a:b] - l2)[:, good].abs().max()) < 1e-10
    assert (d.n_lme_noconv, d.first_lme_noconv) == (noconv, first) and noconv > 0


@pytest.mark.parametrize("precision", [1, 2])
@pytest.mark.parametrize("radius", [1.86, 2.4])
def test_float32_values_do_not_depend_on_the_size(precision, radius):
    """Large calls with float32 grad N give a small call's values bit for bit."""
    from paper_2206_08772_amd.sim import build_neighbors, lme_shape
    x, xp = cloud(N_MP + 37)
    offsets, idx = build_neighbors(x, xp, radius, radius * 1.0001)
    lam, N, dN, _ = lme_shape(x, xp, offsets, idx, 4.0, 1e-14, precision=precision)
    a, b = 64, 64 + 5000
    q0, q1 = int(offsets[a]), int(offsets[b])
    l2, N2, dN2, _ = lme_shape(x, xp[:, a:b].contiguous(), (offsets[a:b + 1] - q0).contiguous(),
                               idx[q0:q1].contiguous(), 4.0, 1e-14, precision=precision)
    for big, small in ((lam[:, a:b], l2), (N[q0:q1], N2), (dN[:, q0:q1], dN2)):
        assert torch.equal(torch.nan_to_num(big), torch.nan_to_num(small))


@pytest.mark.parametrize("precision", ["fp64", "mixed", "mixed_storage"])
@pytest.mark.parametrize("over", [{}, {"kappa": 400.0}])
@pytest.mark.parametrize("skin_h", [0.0, 0.15, 0.3])
def test_kept_lists_give_the_values_of_new_ones(precision, over, skin_h):
    """Rows past 36 pairs are solved in their round after a search and packed
    together with kept lists: the same bits, whatever their share of the rows."""
    w = W.taylor_rod(h=3.2e-3 / 5.8, seed=2, length=16e-3, skin_h=skin_h)
    sim, p = make_sim(w, precision=precision, **over)
    sim.init()
    sim.run(2)
    lam = sim.lam.clone()
    sim.refresh(rebuild=True)
    P = int(sim.offsets[-1])
    rows = torch.diff(sim.offsets)
    assert skin_h == 0.0 or float((rows > 36).double().mean()) > 0.05
    want = [t.clone() for t in (sim.lam, sim.N[:P], sim.dN[:, :P])]
    sums = [sim.m.clone(), sim.f.clone()]
    sim.N[:P] = -1.0
    sim.dN[:, :P] = -1.0
    sim.lam.copy_(lam)
    sim.refresh(rebuild=False)
    for a, b in zip((sim.lam, sim.N[:P], sim.dN[:, :P]), want):
        assert torch.equal(a, b)
    # the sums' order is free: a few hundred terms each
    assert float((sim.m - sums[0]).abs().max()) <= 1e-13 * float(sums[0].max())
    assert float((sim.f - sums[1]).abs().max()) <= 1e-12 * float(sums[1].abs().max())


@pytest.mark.parametrize("precision", ["fp64", "mixed_storage"])
@pytest.mark.parametrize("over", [{}, {"kappa": 400.0}])
@pytest.mark.parametrize("skin_h,order", [(0.0, "morton"), (0.15, "lattice")])
def test_fused_assembly_sums_its_pairs(precision, over, skin_h, order):
    w = W.taylor_rod(h=3.2e-3 / 10.6, seed=2, length=22.4e-3, skin_h=skin_h, hex_order=order)
    assert w.n_mp >= N_MP
    sim, p = make_sim(w, precision=precision, **over)
    sim.init()
    sim.T += 50.0 * torch.rand(w.n_mp, dtype=torch.float64, device="cuda")
    sim.run(2)
    sim.check_diag()
    off = sim.offsets
    P = int(off[-1])
    rows = torch.diff(off)
    assert skin_h == 0.0 or int(rows.max()) > 40
    mp = torch.arange(w.n_mp, device="cuda").repeat_interleave(rows)
    I = sim.idx[:P].long()
    N, g = sim.N[:P], sim.dN[:, :P].double()
    s = sim.sigma.double()[:, mp]
    v = sim.vol[mp]

    def check(got, pair):
        want = torch.zeros_like(got).index_add_(0, I, pair)
        size = torch.zeros_like(got).index_add_(0, I, pair.abs())
        # up to ~200 terms in another order
        assert float(((got - want).abs() - 1e-13 * size).max()) <= 0.0

    check(sim.m, N * sim.mass[mp])
    check(sim.f[0], -v * (s[0] * g[0] + s[3] * g[1] + s[5] * g[2]))
    check(sim.f[1], -v * (s[3] * g[0] + s[1] * g[1] + s[4] * g[2]))
    check(sim.f[2], -v * (s[5] * g[0] + s[4] * g[1] + s[2] * g[2]))
    if "kappa" in over:
        check(sim.heat[0], N * (sim.mass * sim.T)[mp])
        q = sim.qflux[:, mp]
        check(sim.heat[1], v * (q[0] * g[0] + q[1] * g[1] + q[2] * g[2]))
