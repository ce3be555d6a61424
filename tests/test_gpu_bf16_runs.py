"""BF16 pairs in LDS, G by lower-triangle blocks with G_X kept over a run of pairs: one and several blocks per
side, more blocks than waves (G_X not kept), more than 64 strips, either monomer the larger, mixed sizes where X
and the block count change from pair to pair, and enough pairs for runs of more than one.  Two fixed sweeps
without the polish against stored partial blocks (deterministic mode): the same products of the same rounded
operands in another order of FP32 sums, up to 448 terms a product and 200 pairs a monomer, sqrt(9e4) * 2^-24 =
2e-5 of the coupling terms, and a rounding of Tau that falls the other way, 2^-9 of one of at least
16 terms, 1.2e-4; the coupling terms are below a third of the amplitudes."""
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


@pytest.mark.parametrize("dims, cutoff, sizes", [
    ((2, 1, 1), None, [(5, 27), (5, 27)]), ((2, 1, 1), None, [(2, 8), (2, 24)]), ((2, 1, 1), None, [(6, 30), (2, 8)]),
    ((2, 1, 1), None, [(2, 9), (8, 56)]), ((2, 1, 1), None, [(8, 56), (2, 9)]), ((2, 1, 1), None, [(4, 13), (7, 21)]),
    ((3, 3, 2), None, [(2, 24), (5, 27), (4, 9), (6, 30), (3, 17), (5, 27)] * 3),
    ((8, 8, 8), 2.3, [(2, 8), (4, 9), (3, 17), (2, 8)] * 128),
])
def test_matches_stored_partials(ctx, dims, cutoff, sizes):
    p = make_lattice_problem(cubic_sites(*dims), cutoff, sizes=sizes, workload=952, coupling_scale=0.5)
    pid = ctx.upload(p)
    got = []
    for det in (0, 1):
        s = ctx.run(pid, tol=0.0, max_sweeps=2, precision=mc.MCPT_BF16, polish=0, deterministic=det,
                    raise_on_error=False)
        assert s["sweeps"] == 2
        got.append(ctx.energy(pid))
    ctx.release(pid)
    for k in ("e_d2", "e_m2", "t"):
        a, b = np.asarray(got[0][k]), np.asarray(got[1][k])
        assert np.max(np.abs(a - b)) <= RTOL * np.max(np.abs(b)), k
