"""The measured rate of v_mfma_f64_4x4x4: positive and at most the published FP64 matrix peak; the record keeps its
size (the field stands where the padding was)."""
import ctypes

import pytest

import paper_1409_2700_amd as mc


def test_record_keeps_its_size():
    assert ctypes.sizeof(mc.mcpt.mcpt_rates) == 32


@pytest.mark.gpu
def test_rate_is_physical():
    r = mc.device_rates(0)
    print(f"[gpu] rates {r}", flush=True)
    assert 10.0 < r["mfma_f64_4x4x4_tflops"] <= 78.6 * 1.02
