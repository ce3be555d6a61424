"""BF16 pairs in LDS, G by lower-triangle blocks, at the block counts of single pairs: batches of two-monomer
clusters, more pairs than a quarter of the largest grid (with fewer, all of G is formed).  Two fixed sweeps
without the polish against stored partial blocks (deterministic mode): the same products of the same rounded
operands in another order of FP32 sums, at most 448 terms a product, sqrt(448) * 2^-24 = 1e-6 of the coupling
terms, and a rounding of Tau that falls the other way, 2^-9 of one of at least 16 terms, 1.2e-4; the
coupling terms are below a third of the amplitudes."""
import numpy as np
import pytest

from synth import cubic_sites, make_lattice_problem
import paper_1409_2700_amd as mc

pytestmark = pytest.mark.gpu

RTOL = 1e-4


@pytest.fixture(scope="module")
def ctx():
    c = mc.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("a, b", [
    ((5, 27), (5, 27)), ((2, 8), (2, 24)), ((6, 30), (2, 8)), ((2, 9), (8, 56)), ((8, 56), (2, 9)), ((4, 13), (7, 21)),
    ((2, 8), (2, 8)),
])
def test_batches_match_stored_partials(ctx, a, b):
    clusters = 2 * mc.device_rates(0)["compute_units"] + 3   # grids hold at most eight workgroups per compute unit
    probs = [make_lattice_problem(cubic_sites(2, 1, 1), None, sizes=[a, b], workload=970 + k, coupling_scale=0.5)
             for k in range(3)]
    pid = ctx.upload_batch([probs[k % 3] for k in range(clusters)])
    got = []
    for det in (0, 1):
        ctx.run(pid, tol=0.0, max_sweeps=2, precision=mc.MCPT_BF16, polish=0, deterministic=det, raise_on_error=False)
        got.append(ctx.energy(pid))
    ctx.release(pid)
    for k in ("e_d2", "e_m2", "t"):
        x, y = np.asarray(got[0][k]), np.asarray(got[1][k])
        assert np.max(np.abs(x - y)) <= RTOL * np.max(np.abs(y)), k
