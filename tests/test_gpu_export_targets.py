"""T fetched into memory that HIP knows, below and above the size from which ordinary host arrays are filled by
several threads: pinned host memory and device memory hold, bitwise, what an ordinary array gets."""
import ctypes

import numpy as np
import pytest
import torch

from synth import cubic_sites, make_lattice_problem
import paper_1409_2700_amd as mc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(2, 2, 2), (4, 4, 4)], ids=["1MB", "9MB"])
@pytest.mark.parametrize("where", ["pinned", "device"])
def test_t_into_known_memory(dims, where):
    prob = make_lattice_problem(cubic_sites(*dims), 1.1, o=5, v=27, workload=982)
    with mc.Context(0) as ctx:
        pid = ctx.upload(prob)
        ctx.run(pid, tol=0.0, max_sweeps=1)
        want = ctx.energy(pid)["t"]
        kw = dict(pin_memory=True) if where == "pinned" else dict(device="cuda")
        buf = torch.zeros(want.size, dtype=torch.float64, **kw)
        torch.cuda.synchronize()
        print(f"[gpu] T of {want.nbytes} bytes into {where} memory", flush=True)
        st = mc.mcpt.lib().mcpt_energy(ctx.h, pid, None, None, None, ctypes.c_void_p(buf.data_ptr()))
        assert st == mc.MCPT_OK
        assert np.array_equal(buf.cpu().numpy().view(np.uint64), want.view(np.uint64))
