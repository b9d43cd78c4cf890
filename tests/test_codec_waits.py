"""The interest-vector encoder's last workgroup reads what every wave of the
others has written with atomics, and only one thread per workgroup releases it:
in the gfx950 code, each wave waits for its own memory operations (vmcnt(0))
before the barrier that precedes that release."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2001_08250_amd import buildlib

KERNELS = ("codec_count_kernel", "codec_length_kernel", "codec_write_kernel")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_waves_wait_for_their_atomics_before_the_release(tmp_path):
    out = str(tmp_path / "iv_codec.s")
    subprocess.run(["hipcc", *buildlib.COMMON, *buildlib.DEVICE, "--cuda-device-only", "-S",
                    os.path.join(buildlib.CSRC, "iv_codec.hip"), "-o", out], check=True)
    text = open(out).read()
    for name in KERNELS:
        body = re.search(rf"^\S*{name}\S*:.*?s_endpgm", text, re.M | re.S).group(0)
        ops = re.findall(r"^\s+(s_waitcnt[^\n]*|s_barrier|buffer_wbl2[^\n]*|global_(?:atomic|store)\S*)", body, re.M)
        release = next(i for i, op in enumerate(ops) if op.startswith("buffer_wbl2"))
        barrier = max(i for i in range(release) if ops[i] == "s_barrier")
        before = [op for op in ops[:barrier] if not op.startswith("s_waitcnt lgkmcnt")]
        assert before[-1].startswith("s_waitcnt") and "vmcnt(0)" in before[-1], (name, before[-3:])
