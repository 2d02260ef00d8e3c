"""Waves per SIMD of built kernels whose register counts lie at a limit (no GPU needed)."""
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from test_kernel_resources import kernel_metadata  # noqa: E402


def test_two_steps_on_one_wave_of_bkg_in_fp32_keep_four_waves(tmp_path):
    # 512 registers per SIMD lane: four waves up to 128 (FP32, BF16 and FP16 storage, with and
    # without a reference velocity; single case and batch)
    md = {k: v for k, v in kernel_metadata(tmp_path).items()
          if ("step2b_ptr_kernelIf" in k or "batch2_kernelIf" in k) and "Li1E" in k}
    assert len(md) >= 9
    assert all(v["vgpr_count"] <= 128 for v in md.values()), md
