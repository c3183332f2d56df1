"""Private memory of the epilogue's kernels, from the compiler's own listing."""
import os
import re
import subprocess

from paper_2310_03505_amd import build as B


def test_epilogue_uses_no_scratch(tmp_path):
    """Neither form of k_post spills or keeps a value in scratch memory."""
    out = tmp_path / "post.s"
    r = subprocess.run([B.HIPCC, *B.FLAGS, "--cuda-device-only", "-S", os.path.join(B.CSRC, "post.hip"), "-o", str(out)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    kernels = re.findall(r"\.name:\s+(\S*k_post\S*)\n\s+\.private_segment_fixed_size: (\d+)", out.read_text())
    assert len(kernels) == 2
    assert all(int(size) == 0 for _, size in kernels), kernels
