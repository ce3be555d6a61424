"""The FP64 pair kernel with V in LDS, adding to G by atomics, at the sizes where its cuts change: more pairs than a
quarter of the device's compute units (fewer run in the two-launch form instead), as a batch of two-monomer
clusters of three different draws.  Two fixed sweeps and the energy pass against the oracle: every
amplitude and energy within 1e-12 of the largest (sums of at most 448 products of order-one terms differ by
rounding, 448 * 2^-53 = 5e-14)."""
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


@pytest.fixture(scope="module")
def clusters():
    return mc.device_rates(0)["compute_units"] // 4 + 3


@pytest.mark.parametrize("a, b", [
    ((1, 1), (1, 8)), ((1, 7), (3, 3)), ((2, 8), (4, 4)), ((1, 1), (5, 27)), ((8, 56), (3, 7)), ((3, 7), (8, 56)),
    ((3, 8), (3, 9)), ((4, 9), (5, 27)), ((5, 27), (4, 9)), ((5, 11), (4, 15)), ((8, 8), (8, 8)), ((5, 20), (5, 20)),
    ((8, 9), (8, 17)), ((5, 27), (5, 27)), ((5, 27), (8, 18)), ((8, 18), (5, 27)), ((8, 20), (4, 10)), ((8, 56), (4, 9)),
    ((6, 19), (7, 11)),
])
def test_batches_of_two_monomers_match_oracle(ctx, clusters, a, b):
    probs = [make_lattice_problem(cubic_sites(2, 1, 1), None, sizes=[a, b], workload=960 + k, coupling_scale=0.5)
             for k in range(3)]
    want = [mcpt_oracle.solve(p, tol=0.0, max_sweeps=2) for p in probs]
    batch = [probs[k % 3] for k in range(clusters)]
    pid = ctx.upload_batch(batch)
    ctx.run(pid, tol=0.0, max_sweeps=2)
    e = ctx.energy(pid)
    sums = ctx.cluster_results(pid)
    ctx.release(pid)

    def close(got, ref):
        return np.max(np.abs(got - ref)) <= RTOL * np.max(np.abs(ref))

    n_t = len(e["t"]) // clusters
    for q in range(clusters):
        r = want[q % 3]
        assert sums[q]["sweeps"] == 2 and abs(sums[q]["e_total"] - r.e_total) <= RTOL * abs(r.e_total), q
        assert close(e["e_d2"][q:q + 1], r.e_d2) and close(e["e_m2"][2 * q:2 * q + 2], r.e_m2), q
        t = mc.mcpt.split_t(e["t"][q * n_t:(q + 1) * n_t], batch[q].n_occ, batch[q].n_vir)
        for x in range(2):
            assert close(t[x], r.T[x]), (q, x)
