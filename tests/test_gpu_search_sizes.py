"""Support lists against a brute-force float64 search, bit for bit: MP counts at
the edges of a compaction group (64), of a run of counts (16384) and of the direct
path (8192); few cells, whose MPs are split among waves and which the fill scans
itself, and more than one scan workgroup of cells; rows around 32, 40 and 64 ids; capacities that do not fit."""
import numpy as np
import pytest
import torch

from oracle import search as OS
from tests.gpu_common import require_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def check(X, P, r, cell):
    from paper_2206_08772_amd.sim import build_neighbors
    want_off, want = OS.neighbors_bruteforce(X, P, r)
    off, idx = build_neighbors(to_dev(X), to_dev(P), r, cell)
    np.testing.assert_array_equal(off.cpu().numpy(), want_off)
    np.testing.assert_array_equal(idx.cpu().numpy(), want)
    return np.diff(want_off)


@pytest.mark.parametrize("n_mp", [1, 63, 64, 65, 4096, 8191, 8192, 8193, 16383, 16385, 33001])
@pytest.mark.parametrize("r", [0.16, 0.21, 0.7])
def test_sizes(n_mp, r):
    rng = np.random.default_rng(n_mp)
    X = rng.uniform(0, 1, (1500, 3))
    P = rng.uniform(-0.05, 1.05, (n_mp, 3))
    rows = check(X, P, r, r * 1.0001)
    if n_mp > 4000:
        assert rows.max() > (30 if r < 0.2 else 64)
        assert r > 0.5 or rows.min() < 4


@pytest.mark.parametrize("n_nodes", [1, 31, 32, 33, 39, 40, 41, 64, 65])
def test_one_cell_rows_of_one_length(n_nodes):
    rng = np.random.default_rng(n_nodes)
    X = rng.uniform(0, 1, (n_nodes, 3))
    rows = check(X, rng.uniform(0, 1, (333, 3)), 2.0, 2.0)
    assert (rows == n_nodes).all()


@pytest.mark.parametrize("side,n_mp", [(19, 200), (19, 9000), (20, 9000), (27, 9000)])
def test_many_cells(side, n_mp):
    """Cells scanned by the fill, up to near its limit of 8192, by one scan
    workgroup, and by two (27^3 cells of edge 0.98)."""
    rng = np.random.default_rng(5)
    g = np.arange(float(side))
    X = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    X = X + rng.uniform(-0.02, 0.02, X.shape)
    check(X, rng.uniform(-1, side, (n_mp, 3)), 0.97, 0.98)


@pytest.mark.parametrize("n_mp", [65536, 65537])
def test_many_mps_in_few_cells(n_mp):
    rng = np.random.default_rng(n_mp)
    X = rng.uniform(0, 1, (500, 3))
    check(X, rng.uniform(0, 1, (n_mp, 3)), 0.2, 0.21)


@pytest.mark.parametrize("n_mp", [500, 8192, 9000])
def test_lists_that_do_not_fit_are_counted_only(n_mp):
    import ctypes as C
    from paper_2206_08772_amd import _lib
    from paper_2206_08772_amd.sim import Workspace, _ptr, _stream
    rng = np.random.default_rng(n_mp)
    X, P = rng.uniform(0, 1, (700, 3)), rng.uniform(0, 1, (n_mp, 3))
    want_off, want = OS.neighbors_bruteforce(X, P, 0.2)
    xn, xm = to_dev(X), to_dev(P)
    for cap in (0, len(want) - 1, len(want)):
        off = torch.full((n_mp + 1,), -1, dtype=torch.int64, device="cuda")
        idx = torch.full((len(want),), -7, dtype=torch.int32, device="cuda")
        ws = Workspace(700, n_mp, cap, "cuda")
        need = C.c_int64(-1)
        code = _lib.lib().otm_build_neighbors(700, _ptr(xn), n_mp, _ptr(xm), 0.2, 0.2, cap,
                                              _ptr(off), _ptr(idx), C.byref(need), ws.ptr,
                                              ws.nbytes, _stream())
        np.testing.assert_array_equal(off.cpu().numpy(), want_off)
        assert need.value == len(want)
        if cap == len(want):
            assert code == _lib.OTM_OK
            np.testing.assert_array_equal(idx.cpu().numpy(), want)
        else:
            assert code == _lib.OTM_ERR_CAPACITY
            assert (idx == -7).all()


@pytest.mark.parametrize("per_radius,length", [(3.2, 9.6e-3), (5.8, 9.6e-3), (13.0, 24e-3),
                                               (14.0, 26e-3)])
def test_lists_of_a_step(per_radius, length):
    """The step's search, whose box the node update forms for up to 65536 nodes,
    finds what the stand-alone call finds at the new positions."""
    import otm_workloads as W
    from paper_2206_08772_amd.sim import build_neighbors
    from tests.gpu_common import make_sim
    w = W.taylor_rod(h=3.2e-3 / per_radius, seed=2, length=length)
    assert (per_radius < 14) == (len(w.x_nodes) <= 65536)
    sim, p = make_sim(w)
    sim.init()
    sim.du[0] += 0.3 * w.h            # out of the box of the last search
    for _ in range(2):
        sim.step()
        off, idx = build_neighbors(sim.x, sim.xp, p["r_list"], p["cell_size"])
        assert torch.equal(sim.offsets, off)
        assert torch.equal(sim.idx[:idx.numel()], idx)
