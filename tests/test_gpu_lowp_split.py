"""Reduced-precision pairs read from L2, two launches per chunk, at the sizes where its cuts change: one, two, five,
six and more tiles per side, exact and ragged multiples of the tile and of the BF16 chunk, and (many pairs)
several per XCD.  Two fixed sweeps without the polish against the one-launch kernel, which deterministic mode
takes.  Both form the same products of the same rounded operands and differ in the order of
FP32 sums: up to 2500 products, sqrt(2500) * 2^-24 = 3e-6 of the coupling terms, which are below a third of the
amplitudes; in BF16 a rounding of Tau that falls the other way (2^-9) in one of the at least 16 terms of a sum
adds 2^-9 / 16 = 1.2e-4 of them."""
import numpy as np
import pytest

from synth import cubic_sites, make_lattice_problem
import paper_1409_2700_amd as mc

pytestmark = pytest.mark.gpu

RTOL = {mc.MCPT_FP32: 1e-6, mc.MCPT_BF16: 1e-4}


@pytest.fixture(scope="module")
def ctx():
    c = mc.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("precision", [mc.MCPT_FP32, mc.MCPT_BF16], ids=["fp32", "bf16"])
@pytest.mark.parametrize("dims, sizes", [
    ((2, 1, 1), [(8, 56), (8, 56)]), ((2, 1, 1), [(5, 27), (8, 56)]), ((2, 1, 1), [(8, 56), (5, 27)]),
    ((2, 1, 1), [(4, 52), (2, 101)]), ((2, 1, 1), [(2, 40), (8, 70)]), ((2, 1, 1), [(8, 70), (2, 41)]),
    ((2, 1, 1), [(2, 16), (8, 165)]), ((2, 1, 1), [(1, 13), (10, 250)]), ((2, 1, 1), [(6, 21), (7, 60)]),
    ((3, 2, 2), [(8, 28), (7, 33), (8, 28), (6, 37)] * 3),
])
def test_matches_the_one_launch_kernel(ctx, dims, sizes, precision):
    p = make_lattice_problem(cubic_sites(*dims), None, sizes=sizes, workload=951, coupling_scale=0.5)
    pid = ctx.upload(p)
    got = []
    for det in (0, 1):
        s = ctx.run(pid, tol=0.0, max_sweeps=2, precision=precision, polish=0, deterministic=det, raise_on_error=False)
        assert s["sweeps"] == 2
        got.append(ctx.energy(pid))
    ctx.release(pid)
    for k in ("e_d2", "e_m2", "t"):
        a, b = np.asarray(got[0][k]), np.asarray(got[1][k])
        assert np.max(np.abs(a - b)) <= RTOL[precision] * np.max(np.abs(b)), k
