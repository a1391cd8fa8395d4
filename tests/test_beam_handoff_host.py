"""How the beam kernels hand data from many workgroups to the last of them (CPU:
the device code is compiled to assembly and read).

A missing acquire shows on a GPU only now and then and as wrong beams, so the
built code is checked instead: between the ticket (a returning atomic) and the
first agent-scope load of what the other workgroups wrote, the last workgroup
invalidates its caches, and it reads by loads, not by read-modify-writes that the
compiler turns into loads with no ordering of their own.
"""
import os
import re
import subprocess

import pytest

from paper_2608_00938_amd import build

KERNELS = ("topk_select_kernel", "topk_fused_rows_kernel")


@pytest.fixture(scope="module")
def functions(tmp_path_factory):
    """Assembly lines of every kernel that hands data over, by mangled name."""
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc on this host")
    out = str(tmp_path_factory.mktemp("asm") / "beam.s")
    subprocess.run([build.HIPCC, *build.CFLAGS, "--offload-device-only", "-S",
                    os.path.join(build.CSRC, "beam.hip"), "-o", out], check=True, capture_output=True)
    found, name = {}, None
    with open(out) as f:
        for line in f:
            m = re.match(r"(\w+):\s*; @", line)
            if m:
                name = m.group(1) if any(k in m.group(1) for k in KERNELS) else None
                if name:
                    found[name] = []
            elif name and line.startswith("\t") and not line.startswith("\t."):
                found[name].append(line.split(";")[0].strip())
    return found


def test_every_handoff_kernel_is_found(functions):
    for k, n in zip(KERNELS, (5, 4)):
        assert sum(k in name for name in functions) == n, k


def test_last_workgroup_acquires_before_it_reads(functions):
    for name, code in functions.items():
        shared = [i for i, c in enumerate(code) if c.startswith("global_load") and c.endswith("sc1")]
        assert shared, name
        inv = [i for i, c in enumerate(code) if c == "buffer_inv sc1"]
        assert len(inv) == 1 and inv[0] < shared[0], name
        # the ticket's value has arrived before the invalidation, a barrier follows it
        ticket = max(i for i, c in enumerate(code[:inv[0]]) if re.match(r"global_atomic_add .* sc0$", c))
        assert "s_waitcnt vmcnt(0)" in code[ticket:inv[0]], name
        assert "s_barrier" in code[inv[0]:shared[0]], name
        # each wave's own writes are performed before the barrier ahead of the ticket
        before = code[:ticket]
        bar = max(i for i, c in enumerate(before) if c == "s_barrier")
        wait = max(i for i, c in enumerate(before[:bar]) if c == "s_waitcnt vmcnt(0)")
        last_write = max(i for i, c in enumerate(before) if c.startswith("global_atomic"))
        assert last_write < wait < bar, name
