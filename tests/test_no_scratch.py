"""The fp32 FFN's kernels hold 128 registers, four workgroups per CU: none of them may spill to scratch memory, the ones that
sort the assignments included (read from the metadata of the kernels' own build)."""
import os
import re
import subprocess

from paper_2503_06823_amd import build as B


def test_fp32_products_use_no_scratch(tmp_path):
    out = tmp_path / "ffn_f32.s"
    subprocess.run([B._hipcc(), *B.FLAGS, "-S", "--cuda-device-only", os.path.join(B.CSRC, "ffn_f32.hip"), "-o", str(out)], check=True,
                   capture_output=True)
    text = out.read_text()
    kernels = re.findall(r"\.name:\s+(\S*grouped_gemm_f32\S*)\n.*?\.private_segment_fixed_size: (\d+)", text, re.S)
    assert len(kernels) == 10 and any("SortingGather" in name for name, _ in kernels)
    assert [k for k in kernels if k[1] != "0"] == []
