"""Few pairs in two launches, whether they fit LDS or not: clusters on both sides of the rule (a quarter as many pairs
as compute units; the largest pair's size), LDS and L2 pairs together, one tile and ragged sizes, plain and replayed
from a graph.  Three fixed sweeps and the energy pass against the oracle: every amplitude and energy within 1e-12 of
the largest (sums of at most 448 products of order-one terms differ by rounding, 448 * 2^-53 = 5e-14 each)."""
import numpy as np
import pytest

from oracle import mcpt_oracle
from synth import cubic_sites, make_lattice_problem
import paper_1409_2700_amd as mc

pytestmark = pytest.mark.gpu

RTOL = 1e-12


@pytest.fixture(scope="module")
def ctx():
    c = mc.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("dims, sizes", [
    ((2, 2, 2), [(5, 27)] * 8), ((2, 2, 2), [(1, 3), (5, 27), (2, 8), (6, 21), (3, 17), (1, 1), (4, 9), (2, 24)]),
    ((2, 2, 1), [(8, 56), (5, 27), (1, 7), (8, 56)]), ((2, 2, 2), [(3, 21)] * 8), ((2, 2, 2), [(3, 20)] * 8),
    ((11, 1, 1), [(4, 20)] * 11), ((3, 2, 2), [(4, 20)] * 12),
])
def test_matches_oracle(ctx, dims, sizes, graph):
    p = make_lattice_problem(cubic_sites(*dims), None, sizes=sizes, workload=953, coupling_scale=0.5)
    r = mcpt_oracle.solve(p, tol=0.0, max_sweeps=3)
    pid = ctx.upload(p)
    for _ in range(2):   # the second run has the task lists
        s = ctx.run(pid, tol=0.0, max_sweeps=3, graph=graph, raise_on_error=False)
        e = ctx.energy(pid)
        assert s["sweeps"] == 3
        assert np.max(np.abs(e["e_d2"] - r.e_d2)) <= RTOL * np.max(np.abs(r.e_d2))
        assert np.max(np.abs(e["e_m2"] - r.e_m2)) <= RTOL * np.max(np.abs(r.e_m2))
        for x, t in enumerate(mc.mcpt.split_t(e["t"], p.n_occ, p.n_vir)):
            assert np.max(np.abs(t - r.T[x])) <= RTOL * np.max(np.abs(r.T[x])), x
    ctx.release(pid)
