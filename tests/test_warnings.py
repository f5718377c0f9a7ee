"""Every source passes the compiler's front end without a warning, for the device and for the host."""
import os
import re
import subprocess

import pytest

from paper_2406_11235_amd import build


@pytest.mark.parametrize("source", build.SOURCES)
def test_no_warnings(source):
    flags = [f for f in build.FLAGS if f != "-shared"]
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags + ["-fsyntax-only", "-x", "hip", os.path.join(build.CSRC, source)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    # (the host pass does not know the device's features, and says so in lines of another form)
    assert res.returncode == 0 and not re.findall(r".*: warning: .*", res.stderr), res.stderr[-4000:]
