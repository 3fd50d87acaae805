"""bench.py goes by the kernel that ran (no GPU)."""
import os
import sys
import types

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402

SPEC = types.SimpleNamespace(cells=400 * 400, q=512, nx=400, ny=400, n_azim=32)


@pytest.mark.parametrize("form,kernel,dtype", [("banded", "banded_euler_kernel<2, 1024, 0, 0>", "f32"),
                                               ("banded", "banded_euler_kernel<2, 1024, 1, 0>", "bf16"),
                                               ("fused", "sparse_step_kernel<0, 0, 1024>", "f32"),
                                               ("fused", "sparse_step_kernel<2, 0, 512>", "f16"),
                                               ("separate", "sparse_step_kernel<0, 0, 512>", "f32")])
def test_steps_on_the_vector_units_are_named_and_rated_so(form, kernel, dtype):
    res = {"form": form, "kernel": kernel, "kms": {"contraction": 0.4, "stream_collide": 0.0}, "chunk": 4,
           "work": {"nonzero_flops": 1e9, "tile_flops": 6e9, "dense_flops": 9e9}}
    r = bench.roofline(res, SPEC, dtype)
    assert r["kernel"] == kernel and r["kernel_ms"] == pytest.approx(0.4)
    assert r["compute_peak_TFLOPs"] == bench.PEAK_FP32_VALU_TFLOPS
    # no rate of blocks that no kernel multiplied
    assert r["executed_over_nonzero"] is None and r["kernels"] == {}


@pytest.mark.parametrize("form,kernel,dtype,peak", [("fused", "gemm_f32_kernel<true>", "f32", 157.3),
                                                    ("fused", "gemm_lp_kernel<1, true>", "bf16", 2500.0)])
def test_tile_contractions_are_rated_on_the_matrix_cores(form, kernel, dtype, peak):
    res = {"form": form, "kernel": kernel, "kms": {"contraction": 0.4, "stream_collide": 0.0}, "chunk": 4,
           "work": {"nonzero_flops": 1e9, "tile_flops": 6e9, "dense_flops": 9e9}}
    r = bench.roofline(res, SPEC, dtype)
    assert r["kernel"] == kernel and r["compute_peak_TFLOPs"] == peak
    assert r["kernels"]["contraction"]["executed_TFLOPs"] == pytest.approx(6e9 / 0.4e-3 / 1e12)


def test_separate_kernels_are_named_by_the_slower():
    res = {"form": "separate", "kernel": "gemm_f32_kernel<false>", "chunk": 4,
           "kms": {"contraction": 0.2, "stream_collide": 0.3},
           "work": {"nonzero_flops": 1e9, "tile_flops": 6e9, "dense_flops": 9e9}}
    assert bench.roofline(res, SPEC, "f32")["kernel"] == "stream_collide_flat_kernel<false>"
    res["kms"]["contraction"] = 0.4
    assert bench.roofline(res, SPEC, "f32")["kernel"] == "gemm_f32_kernel<false>"
