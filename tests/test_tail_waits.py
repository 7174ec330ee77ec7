"""How long a workgroup of recip_tail_kernel waits for the others before it leaves: the rule itself, compiled for the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAIN = """
#include <stdio.h>
#include "%s/paper_2503_10017_amd/csrc/fnn_kernels.hpp"
int main() {
    long long n, m, seeds;
    while (scanf("%%lld %%lld %%lld", &n, &m, &seeds) == 3) printf("%%llu\\n", (unsigned long long)fnn::tail_most_polls(n, m, seeds));
}
"""
LOOK_NS = 130.0                        # an atomic load past the compute unit's cache and 64 cycles of sleep, at the least (133.6 measured)
BLOCK_NS = 18.75 * 32 / 4              # the dearest 32x32 block of scores (fp32 products of 32 channels), on the four SIMDs of one workgroup
SHAPES = [(1, 1, 1), (64 * 48, 64 * 48, 48), (512 * 384, 512 * 384, 3072), (1024 * 768, 1024 * 768, 12288),
          (1024 * 768, 1024 * 768, 1024 * 768), (4096 * 3072, 4096 * 3072, 4096 * 3072), (1, 2**31 - 64, 2**31 - 64), (2**31 - 64,) * 3]


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_a_wait_outlasts_a_phase_that_one_workgroup_does_alone(tmp_path):
    src, exe = tmp_path / "main.cpp", tmp_path / "main"
    src.write_text(MAIN % ROOT)
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", str(src), "-o", str(exe)], check=True, capture_output=True, timeout=300)
    text = "\n".join("%d %d %d" % s for s in SHAPES)
    looks = [int(x) for x in subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True, timeout=60).stdout.split()]
    assert len(looks) == len(SHAPES)
    for (n, m, seeds), got in zip(SHAPES, looks):
        blocks = -(-max(n, m) // 32) * -(-seeds // 32)
        assert got * LOOK_NS > 20 * (blocks * BLOCK_NS + seeds * 2000.0), (n, m, seeds)
        assert got < 2**62
    assert looks[0] < 1.1 * 2**26      # and no longer than it has to be
