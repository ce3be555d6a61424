"""A request with a non-finite integral that is alone in its batch: its one cluster is stopped before
the first sweep, so the solve ends there.  The request fails with MCPT_ERR_NONFINITE in every form of the
solve, and the next request is served as usual."""
import numpy as np
import pytest

from synth import make_workload
import paper_1409_2700_amd as mc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["v", "k"])
@pytest.mark.parametrize("opts", [
    dict(), dict(graph=1), dict(deterministic=1), dict(tol=0.0, max_sweeps=3, graph=1),
    dict(precision=mc.MCPT_FP32), dict(precision=mc.MCPT_FP32, graph=1), dict(precision=mc.MCPT_FP32, polish=0),
    dict(precision=mc.MCPT_BF16), dict(precision=mc.MCPT_BF16, graph=1), dict(precision=mc.MCPT_BF16, max_sweeps=2),
], ids=lambda o: "-".join(f"{k}{v}" for k, v in o.items()) or "fp64")
def test_lone_nonfinite_request_fails(opts, where):
    good = make_workload("hf-2x2x2")
    bad = make_workload("hf-2x2x2")
    setattr(bad, where, getattr(bad, where).copy())
    getattr(bad, where)[5] = np.inf
    opts = {"tol": 1e-10, **opts}
    print(f"[gpu] lone non-finite {where} {opts}", flush=True)
    with mc.Context(0) as ctx:
        ctx.serve_config(workers=1, max_batch=8)
        t = ctx.submit(bad, **opts)
        s = ctx.wait(t, 20000)
        assert s is not None and s["status"] == mc.MCPT_ERR_NONFINITE
        with pytest.raises(mc.MCPTError):
            ctx.energy(t)
        s = ctx.wait(ctx.submit(good, **{**opts, "tol": 1e-10, "max_sweeps": 100}), 20000)
        assert s is not None and s["status"] in (mc.MCPT_OK, mc.MCPT_ERR_NOT_CONVERGED)
