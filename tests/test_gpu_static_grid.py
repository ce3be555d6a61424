"""mcpt_run_static where the LDS variant's slots are near the largest they get (o8v17 and o8v18: 136 x 144 blocks,
Tau and its transpose) and there are more pairs than compute units, so every workgroup's slot is in use, alone and
next to pairs read from L2 whose slots are larger and fewer.  Fixed sweeps against mcpt_run: every result within
1e-12 of the largest (the two differ by the order of the FP64 additions, at most 26 neighbours x 448 products)."""
import numpy as np
import pytest

from synth import cubic_sites, make_lattice_problem
import paper_1409_2700_amd as mc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("large", [0, 1], ids=["lds", "lds-and-l2"])
def test_static_equals_run_with_every_slot_in_use(large):
    n = 64
    sizes = [(8, 17) if k % 2 else (8, 18) for k in range(n)]
    for k in range(large):
        sizes[21 + k] = (8, 56)
    prob = make_lattice_problem(cubic_sites(4, 4, 4), 2, sizes=sizes, workload=953, coupling_scale=0.1)
    assert prob.n_pair > 256
    with mc.Context(0) as ctx:
        pid = ctx.upload(prob)
        out = []
        for run in (ctx.run, ctx.run_static):
            s = run(pid, tol=0.0, max_sweeps=2)
            out.append((s, ctx.energy(pid)))
    (a, ea), (b, eb) = out
    assert a["sweeps"] == b["sweeps"] == 2
    assert abs(a["e_total"] - b["e_total"]) <= 1e-12 * abs(a["e_total"])
    for key in ("e_m2", "e_d2", "t"):
        assert np.max(np.abs(ea[key] - eb[key])) <= 1e-12 * np.max(np.abs(ea[key])), key
