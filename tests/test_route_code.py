"""What the compiler is told about the routing kernels, read from the intermediate code of a device-only compilation."""
import os
import re
import subprocess

from paper_2510_15620_amd import build as B


def test_lanes_of_a_wavefront_meet_between_the_steps_of_the_sort(tmp_path):
    """Steps of the sort inside a wavefront are separated by fences, which order memory but do not make lanes that took
    different sides of the exchange meet again: between the release and the acquire of every such pair stands the wavefront's
    barrier, an operation that all lanes reach together."""
    out = str(tmp_path / "prune.ll")
    subprocess.run([B.HIPCC, *B.COMMON, *B.EXTRA["prune.hip"], "--cuda-device-only", "-S", "-emit-llvm", os.path.join(B.CSRC, "prune.hip"), "-o", out],
                   check=True, capture_output=True)
    lines = [l.strip() for l in open(out)]
    fences = [i for i, l in enumerate(lines) if re.match(r'fence syncscope\("wavefront"\)', l)]
    assert fences and len(fences) % 2 == 0
    for a, b in zip(fences[::2], fences[1::2]):
        assert lines[a].endswith("release") and lines[b].endswith("acquire")
        assert any("@llvm.amdgcn.wave.barrier()" in l for l in lines[a + 1:b]) and not any(re.match(r"br |store |.*= load ", l) for l in lines[a + 1:b])
