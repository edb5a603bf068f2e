"""bench.py: each kernel is held against the ceiling of the form it computes in, nominal and measured."""
import pytest

import bench


@pytest.mark.parametrize("kernel,key", [("gemm_f32x2_128x128", "mfma_f32x2"), ("gemm_f32x3_nt_128x64", "mfma_f32x3"),
                                        ("gemm_f32x3_tn_256x256", "mfma_f32x3"), ("gemm_f32_tn_128x64", "mfma_f32"),
                                        ("gemm_bf16_dl_nt_256x256", "mfma_bf16"), ("tripG_mfma_fwd", "mfma_bf16"),
                                        ("tripD_fwd", "alu_f32"), ("reduce_parts", "hbm")])
def test_ceiling_of_a_kernel(kernel, key):
    assert bench.peak_key(kernel) == key
    nominal = {"copy_GBps": 8000.0, "mfma_f32_TFLOPs": 157.3, "mfma_bf16_TFLOPs": 2500.0}
    # a card that reaches the nominal rates has the same fractions of both
    assert key == "alu_f32" or abs(bench.measured_rates(nominal)[key] / bench.PEAK[key][0] - 1.0) < 1e-3
