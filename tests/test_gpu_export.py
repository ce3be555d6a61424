"""Large results on their way to the host: T below and above the size from which the array is
fetched in parts by several threads (one chunk a part, and several with a rest), against the same
clusters fetched one by one; the pair amplitudes of the dimer-internal terms against the oracle,
and that fetching them changes no later solve."""
import numpy as np
import pytest

from oracle import mcpt_dimer
from synth import make_lattice_problem
from synth.hf_lattice import cubic_sites, dimer_integrals, lccd_integrals
import paper_1409_2700_amd as mc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = mc.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("dims,copies", [((3, 3, 3), 1), ((3, 3, 3), 2), ((4, 4, 4), 6)])
def test_t_in_parts_equals_one_by_one(ctx, dims, copies):
    probs = [make_lattice_problem(cubic_sites(*dims), 1.1, o=5, v=27, workload=980, cluster=q) for q in range(copies)]
    opts = dict(tol=0.0, max_sweeps=2, deterministic=1)
    pid = ctx.upload_batch(probs)
    ctx.run(pid, raise_on_error=False, **opts)
    t = ctx.energy(pid)["t"]
    ctx.release(pid)
    at = 0
    for p in probs:   # 3.9 MB (fetched whole) or 9.3 MB (in parts of one chunk) each
        sid = ctx.upload(p)
        ctx.run(sid, raise_on_error=False, **opts)
        one = ctx.energy(sid)["t"]
        ctx.release(sid)
        assert np.array_equal(t[at:at + one.size].view(np.uint64), one.view(np.uint64))
        at += one.size
    assert at == t.size


def test_dimer_tau_in_parts(ctx):
    p = make_lattice_problem(cubic_sites(3, 3, 3), 1.1, o=5, v=27, workload=981)   # 54 pairs, 7.9 MB
    ints, dints = lccd_integrals(p), dimer_integrals(p)
    ref = mcpt_dimer.solve(p, ints, dints, tol=0.0, max_sweeps=2)
    pid = ctx.upload(p)
    ctx.lccd_attach(pid, ints)
    ctx.dimer_attach(pid, dints)
    opts = dict(tol=0.0, max_sweeps=2)
    assert ctx.run(pid, raise_on_error=False, **opts)["return"] in (mc.MCPT_OK, mc.MCPT_ERR_NOT_CONVERGED)
    tau, t = ctx.dimer_tau(pid), ctx.energy(pid)["t"]
    assert ctx.run(pid, raise_on_error=False, **opts)["return"] in (mc.MCPT_OK, mc.MCPT_ERR_NOT_CONVERGED)
    again, t2 = ctx.dimer_tau(pid), ctx.energy(pid)["t"]
    ctx.release(pid)
    want = np.concatenate([np.asarray(x).ravel() for x in ref.Tau])
    assert np.abs(tau - want).max() <= 1e-10 * np.abs(want).max()
    # G is summed in any order: rounding, where a changed source would show in the second digit
    assert np.abs(tau - again).max() <= 1e-12 * np.abs(want).max()
    assert np.abs(t - t2).max() <= 1e-12 * np.abs(t).max()
