"""The FP64 pair kernel with V in LDS at the sizes where its cuts change: single 8 x 8
blocks, exact and ragged multiples of 8, segments of one to five blocks, more and fewer
tasks than waves, and the largest pair that fits next to one that does not.  Two
monomers, two fixed sweeps and the energy pass against the oracle: every amplitude and
energy within 1e-12 of the largest (sums of at most 448 products of order-one terms
differ by rounding, 448 * 2^-53 = 5e-14), with atomics and with stored partial blocks."""
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


@pytest.mark.parametrize("det", [0, 1])
@pytest.mark.parametrize("a, b", [
    ((1, 1), (1, 8)), ((1, 7), (3, 3)), ((2, 8), (4, 4)), ((1, 1), (5, 27)), ((8, 56), (3, 7)), ((3, 7), (8, 56)),
    ((4, 9), (5, 27)), ((5, 27), (4, 9)), ((8, 8), (8, 8)), ((5, 20), (5, 20)), ((8, 17), (8, 17)), ((5, 27), (5, 27)),
    ((5, 27), (8, 18)), ((8, 18), (5, 27)), ((8, 20), (4, 10)), ((8, 56), (4, 9)), ((6, 19), (7, 11)),
])
def test_two_monomers_match_oracle(ctx, a, b, det):
    p = make_lattice_problem(cubic_sites(2, 1, 1), None, sizes=[a, b], workload=950, coupling_scale=0.5)
    r = mcpt_oracle.solve(p, tol=0.0, max_sweeps=2)
    pid = ctx.upload(p)
    s = ctx.run(pid, tol=0.0, max_sweeps=2, deterministic=det)
    e = ctx.energy(pid)
    ctx.release(pid)
    assert s["sweeps"] == 2

    def close(got, want):
        return np.max(np.abs(got - want)) <= RTOL * np.max(np.abs(want))

    assert close(e["e_d2"], r.e_d2) and close(e["e_m2"], r.e_m2)
    assert abs(s["e_total"] - r.e_total) <= RTOL * abs(r.e_total)
    for x, t in enumerate(mc.mcpt.split_t(e["t"], p.n_occ, p.n_vir)):
        assert close(t, r.T[x]), x
