"""How bench.py prices the kernels it times."""
import pytest

import bench
import workloads
from paper_2507_05829_amd import lop


@pytest.mark.parametrize("kernel,dtype,peak", [
    ("conv_patch_kernel_bands<float, 64, 32, false, 1>", "f32", 2500 / 6),
    ("conv_gemm_split_kernel<32, 64, 1, 2>", "f32", 2500 / 6),
    ("conv_stem_pool_kernel_bands<float, 1>", "f32", 2500 / 6),
    ("conv_narrow_patch_kernel_bands<float, 9, 81920>", "f32", 157.3),
    ("conv_gemm_kernel<float, 128, 128, 2, 2, 2>", "f32", 157.3),
    ("conv_patch_kernel<__bf16, 128, 64, false, 1>", "bf16", 2500),
])
def test_kernels_are_priced_on_the_instructions_they_run_on(kernel, dtype, peak):
    assert bench.mfma_peak(kernel, dtype) == pytest.approx(peak)
    group = dict(name=kernel, launches=1, total_us=10.0, avg_us=10.0, tflops=75.0, gbs=1.0, _flop=7.5e8, _bytes=1e4)
    roof = bench.dominant_roofline([group], dtype, "none")
    assert roof["bound"] == "mfma" and roof["frac"] == pytest.approx(75.0 / peak, abs=1e-4)


@pytest.mark.gpu
def test_names_of_kernels_that_multiply_in_parts():
    """The fp32 backbone's kernels, as a plan names them, are found by bench.PARTS."""
    chain = workloads.CONFIGS["resnet18"]()
    plan = lop.Plan(chain, workloads.make_tensors(chain), flags=lop.LOP_FLAG_BATCH_BANDS)
    try:
        names = {plan.layer_kernel(0, l)[0] for l in range(plan.n_layers)} - {""}
    finally:
        plan.destroy()
    parts = {n for n in names if bench.mfma_peak(n, "f32") > 400}
    assert {n.split("<")[0] for n in parts} == {"conv_stem_pool_kernel_bands", "conv_patch_kernel_bands"}, names
    assert any(n.startswith("conv_narrow_patch_kernel") for n in names - parts)
