"""The tuner on a problem without a pair in LDS, where it times the one-launch kernel: the shape with the least time
is chosen, and the solves that do not use the choice (two launches) and those that do (deterministic) both
reach the FP64 energies afterwards."""
import pytest

from synth import cubic_sites, make_lattice_problem
import paper_1409_2700_amd as mc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [mc.MCPT_FP32, mc.MCPT_BF16], ids=["fp32", "bf16"])
def test_solves_after_tuning_pairs_read_from_l2(prec):
    prob = make_lattice_problem(cubic_sites(3, 3, 3), 2, o=8, v=56, workload=983, coupling_scale=0.05)
    with mc.Context(0) as ctx:
        pid = ctx.upload(prob)
        ref = ctx.run(pid, tol=1e-10)
        rep = ctx.autotune(pid, prec)
        ms = [v["ms"] for v in rep["variants"]]
        print("[gpu] shapes, ms: " + " ".join(f"{m:.3f}" for m in ms), flush=True)
        assert ms[rep["best"]] == min(ms) > 0.0
        for det in (0, 1):
            s = ctx.run(pid, tol=1e-10, precision=prec, deterministic=det)
            assert abs(s["e_total"] - ref["e_total"]) <= 1e-10 * abs(ref["e_total"])
