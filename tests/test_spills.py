"""The quantizer's kernels, whose loops live in registers, spill no more of them than they are known to."""
import os
import re
import subprocess

from paper_2406_11235_amd import build

# (kernel, kV, V, code): registers
KNOWN = {("forward", 2, 1, 5): 33, ("forward", 3, 1, 5): 28, ("forward", 4, 1, 5): 25, ("forward", 4, 2, 2): 28,
         ("forward", 4, 2, 3): 28, ("forward", 8, 2, 2): 36, ("forward", 8, 2, 3): 36, ("few", 2, 1, 0): 1, ("few", 2, 1, 1): 1}


def test_quantizer_spills(tmp_path):
    flags = [f for f in build.FLAGS if f != "-shared"]
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags + [
        "-Rpass-analysis=kernel-resource-usage", "--cuda-device-only", "-x", "hip", "-c",
        os.path.join(build.CSRC, "qtip_viterbi.hip"), "-o", str(tmp_path / "viterbi.o")]
    report = subprocess.run(cmd, capture_output=True, text=True, check=True).stderr
    seen = {}
    for block in report.split("Function Name: ")[1:]:
        kernel = re.match(r"\S*viterbi_(forward|few)_kernelILi(\d)ELi(\d)ELi(\d)E", block)
        if kernel:
            spill = int(re.search(r"VGPRs Spill: (\d+)", block).group(1))
            seen[(kernel.group(1), *map(int, kernel.groups()[1:]))] = spill
    assert len([k for k in seen if k[0] == "forward"]) == 18 and len([k for k in seen if k[0] == "few"]) == 11, sorted(seen)
    assert {k: v for k, v in seen.items() if v > KNOWN.get(k, 0)} == {}
