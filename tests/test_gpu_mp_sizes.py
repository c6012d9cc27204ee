"""The material-point pass's gather against sums of the step's own pairs, for
bodies whose workgroups take from their fewest MPs to their most, with partial
last workgroups and rows past the pipelined slots."""
import pytest
import torch

import otm_workloads as W
from tests.gpu_common import make_sim, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("precision", ["fp64", "mixed", "mixed_storage"])
@pytest.mark.parametrize("per_radius,length,skin_h,rounds",
                         [(3.2, 9.6e-3, 0.0, 4), (5.8, 15e-3, 0.3, 4), (6.9, 22e-3, 0.0, 10),
                          (7.9, 20e-3, 0.3, 12), (8.9, 24e-3, 0.0, 16)])
def test_gather(precision, per_radius, length, skin_h, rounds):
    w = W.taylor_rod(h=3.2e-3 / per_radius, seed=2, length=length, skin_h=skin_h)
    n = w.n_mp
    even = -(-n // 8192) * 2                 # rounds of 16 MPs, one on each of 256 CUs
    assert min(max(even, 4), 16) == rounds
    sim, p = make_sim(w, precision=precision)
    sim.init()
    sim.run(2)
    off, P = sim.offsets.clone(), int(sim.offsets[-1])
    rows = torch.diff(off)
    assert skin_h == 0.0 or int(rows.max()) > 40
    mp = torch.arange(n, device="cuda").repeat_interleave(rows)
    I, N, g = sim.idx[:P].long(), sim.N[:P].clone(), sim.dN[:, :P].double().clone()
    vol = sim.vol.clone()
    sim.step()
    sim.check_diag()
    want, size = torch.zeros(3, n, device="cuda", dtype=torch.float64), 0.0
    want.index_add_(1, mp, N * sim.x[:, I])
    size = float(sim.x.abs().max())
    # up to 60 terms of weights that sum to one, twice rounded each
    assert float((sim.xp - want).abs().max()) <= 1e-14 * size
    H = torch.zeros(3, 3, n, device="cuda", dtype=torch.float64)
    for i in range(3):
        H[i].index_add_(1, mp, sim.du[i, I] * g)
    F = H.permute(2, 0, 1) + torch.eye(3, device="cuda", dtype=torch.float64)
    terms = torch.zeros(n, device="cuda", dtype=torch.float64)
    terms.index_add_(0, mp, sim.du[:, I].abs().sum(0) * g.abs().sum(0))
    assert float(((sim.vol / vol - torch.linalg.det(F)).abs() - 1e-14 * (1 + terms)).max()) <= 0.0


@pytest.mark.parametrize("precision", ["fp64", "mixed_storage"])
@pytest.mark.parametrize("skin_h", [0.05, 0.1, 0.2, 0.35])
def test_tails_of_a_large_body(precision, skin_h):
    """Rows past 32 pairs, from a few to nearly all of them, most with up to 8
    pairs past, the longest with more."""
    w = W.taylor_rod(h=3.2e-3 / 8.9, seed=2, length=24e-3, skin_h=skin_h)
    sim, p = make_sim(w, precision=precision)
    sim.init()
    sim.run(2)
    off, P = sim.offsets.clone(), int(sim.offsets[-1])
    rows = torch.diff(off)
    past = rows[rows > 32] - 32
    assert len(past) > 100 and (skin_h < 0.3 or int(past.max()) > 9)
    mp = torch.arange(w.n_mp, device="cuda").repeat_interleave(rows)
    I, N, g = sim.idx[:P].long(), sim.N[:P].clone(), sim.dN[:, :P].double().clone()
    vol = sim.vol.clone()
    sim.step()
    sim.check_diag()
    want = torch.zeros(3, w.n_mp, device="cuda", dtype=torch.float64)
    want.index_add_(1, mp, N * sim.x[:, I])
    assert float((sim.xp - want).abs().max()) <= 1e-14 * float(sim.x.abs().max())
    H = torch.zeros(3, 3, w.n_mp, device="cuda", dtype=torch.float64)
    for i in range(3):
        H[i].index_add_(1, mp, sim.du[i, I] * g)
    F = H.permute(2, 0, 1) + torch.eye(3, device="cuda", dtype=torch.float64)
    terms = torch.zeros(w.n_mp, device="cuda", dtype=torch.float64)
    terms.index_add_(0, mp, sim.du[:, I].abs().sum(0) * g.abs().sum(0))
    assert float(((sim.vol / vol - torch.linalg.det(F)).abs() - 1e-14 * (1 + terms)).max()) <= 0.0
