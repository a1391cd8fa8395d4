"""How many queries a wave of the bf16 cross-attention kernels loads (CPU: the
device code is compiled to assembly and read).

A wave owns 32 beams per block and reads those rows only; what else it loads is a
neighbour's and delays its first product.  The query loads are the direct-to-LDS
loads with the streaming hint, 64 lanes of 16 bytes each.
"""
import os
import re
import subprocess

import pytest

from paper_2608_00938_amd import build


@pytest.fixture(scope="module")
def query_loads(tmp_path_factory):
    """Query loads per kernel: {(kernel, head dim, beam blocks per wave): count}."""
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc on this host")
    out = str(tmp_path_factory.mktemp("asm") / "cross.s")
    subprocess.run([build.HIPCC, *build.CFLAGS, "--offload-device-only", "-S",
                    os.path.join(build.CSRC, "cross_attn.hip"), "-o", out], check=True, capture_output=True)
    found, key = {}, None
    with open(out) as f:
        for line in f:
            if re.match(r"\w+:\s*; @", line):
                m = re.search(r"cross_attn_bf16_(split_)?kernelILi(\d+)E(?:Li(\d+)E)?", line)
                key = ("split" if m[1] else "whole", int(m[2]), int(m[3] or 1)) if m else None
                if key:
                    found[key] = 0
            elif key and re.match(r"\tglobal_load_lds_dwordx4 .* nt", line):
                found[key] += 1
    return found


def test_a_wave_loads_the_queries_of_its_own_beams(query_loads):
    assert set(query_loads) == {("whole", 32, 1), ("whole", 32, 2), ("whole", 64, 1), ("whole", 64, 2),
                                ("whole", 128, 1), ("split", 32, 1), ("split", 64, 1), ("split", 128, 1)}
    for (kernel, d, blocks), n in query_loads.items():
        assert n * 64 * 16 == 32 * blocks * d * 2, (kernel, d, blocks)
