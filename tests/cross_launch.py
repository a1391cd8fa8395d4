"""Which cross-attention kernel a call takes, by the launch rule of
csrc/cross_attn.hip with the limits read from there, so that a test that means
to reach one of them notices when its sizes no longer do."""
import os
import re

from paper_2608_00938_amd import build

with open(os.path.join(build.CSRC, "cross_attn.hip")) as _f:
    _SRC = _f.read()
_CUS = int(re.search(r"constexpr int kCus = (\d+);", _SRC)[1])
_PER_CU = [int(x) for x in re.search(
    r"constexpr int kSplitPerCu = D == 32 \? (\d+) : \(D == 64 \? (\d+) : (\d+)\);", _SRC).groups()]
_F32_GRID = int(re.search(r"ns < kF32Waves && .*\(128 / ns\)\) < (\d+)\) ns \*= 2;", _SRC)[1])


def bf16_kernel(B, M, H, d):
    """"split" (keys over a workgroup's waves), "half" (128 beams per workgroup) or
    "whole" (256, or 128 at d = 128)."""
    if B * H * -(-M // 32) <= _CUS * _PER_CU[(32, 64, 128).index(d)]:
        return "split"
    if d != 128 and (M <= 128 or B * H * -(-M // 128) <= _CUS):
        return "half"
    return "whole"


def f32_splits(B, M, H):
    """Waves that share a beam group's keys: 4, 2 or 1."""
    ns = 1
    while ns < 4 and B * H * -(-M // (128 // ns)) < _F32_GRID:
        ns *= 2
    return ns
