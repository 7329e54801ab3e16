"""The kernel that adds the pieces of tiles cut along K is built for the arrangements that can be cut, those with 128 weight rows, and
for no other, which nothing would launch (read from the assembly of the kernels' own build)."""
import os
import re
import subprocess

from paper_2503_06823_amd import build as B


def test_fixups_of_arrangements_that_are_cut_only(tmp_path):
    out = tmp_path / "mid.s"
    subprocess.run([B._hipcc(), *B.FLAGS, "-S", "--cuda-device-only", os.path.join(B.CSRC, "ffn_bf16_mid.hip"), "-o", str(out)], check=True,
                   capture_output=True)
    found = re.findall(r"^_ZN4emoe\S*mid_fixupILi(\d)ELi(\d+)ELi(\d+)E\S*:", out.read_text(), re.M)
    # epilogue, token rows, weight rows; SwiGLU (1) takes 128 token rows only
    assert sorted(tuple(map(int, f)) for f in found) == [(0, 64, 128), (0, 128, 128), (1, 128, 128), (2, 64, 128), (2, 128, 128)]
