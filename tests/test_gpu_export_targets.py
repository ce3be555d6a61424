"""T fetched into memory that HIP knows, below and above the size from which ordinary host arrays are filled by
several threads: pinned host memory and device memory hold, bitwise, what an ordinary array gets."""
import ctypes
import os

import numpy as np
import pytest

from synth import cubic_sites, make_lattice_problem
import paper_1409_2700_amd as mc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(2, 2, 2), (4, 4, 4)], ids=["1MB", "9MB"])
@pytest.mark.parametrize("where", ["pinned", "device"])
def test_t_into_known_memory(dims, where):
    prob = make_lattice_problem(cubic_sites(*dims), 1.1, o=5, v=27, workload=982)
    with mc.Context(0) as ctx:
        hip = ctypes.CDLL(os.path.join("/opt/rocm/lib", "libamdhip64.so"))   # the library's runtime
        pid = ctx.upload(prob)
        ctx.run(pid, tol=0.0, max_sweeps=1)
        want = ctx.energy(pid)["t"]
        got = np.zeros_like(want)
        p, size = ctypes.c_void_p(), ctypes.c_size_t(want.nbytes)
        print(f"[gpu] T of {want.nbytes} bytes into {where} memory", flush=True)
        if where == "pinned":
            assert hip.hipHostMalloc(ctypes.byref(p), size, 0) == 0
        else:
            assert hip.hipMalloc(ctypes.byref(p), size) == 0
        try:
            assert mc.mcpt.lib().mcpt_energy(ctx.h, pid, None, None, None, p) == mc.MCPT_OK
            if where == "pinned":
                ctypes.memmove(got.ctypes.data, p, want.nbytes)
            else:
                assert hip.hipMemcpy(got.ctypes.data_as(ctypes.c_void_p), p, size, 2) == 0
        finally:
            (hip.hipHostFree if where == "pinned" else hip.hipFree)(p)
        assert np.array_equal(got.view(np.uint64), want.view(np.uint64))
