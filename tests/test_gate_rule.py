"""The host rule that picks the gate for a problem (one kernel that evaluates
every logit, or the certified filter), against measured times of both on an
MI355X: the faster one at each of these sizes, where they differ by a tenth or
more."""
import os
import re

import pytest

from paper_2609_21483_amd import build as BLD
from tests.cases import gate_filtered, gate_kernel_of

# (T, H, E, k): us of the one-kernel gate, of the filter; sizes at, just above
# and between the steps of the gate's time (whole rounds of workgroups)
MEASURED = [
    ((4096, 4096, 66, 1), 73, 99), ((8192, 4096, 128, 4), 92, 129), ((8200, 4096, 66, 1), 158, 99),
    ((8200, 4096, 128, 4), 156, 130), ((8200, 4096, 128, 8), 158, 138), ((10000, 2048, 100, 1), 83, 64),
    ((12300, 4096, 128, 2), 157, 125), ((20000, 1024, 66, 4), 74, 66), ((16400, 4096, 128, 4), 230, 170),
    ((30000, 1024, 100, 2), 87, 77), ((32800, 4096, 128, 8), 370, 309), ((512, 4096, 128, 8), 50, 124),
    ((16384, 8192, 128, 2), 307, 360), ((12300, 16384, 128, 1), 596, 966), ((4096, 16384, 128, 3), 270, 775),
    ((4096, 4096, 256, 8), 98, 248), ((8192, 2048, 256, 8), 90, 222), ((10000, 4096, 130, 2), 239, 177),
    ((16384, 4096, 192, 3), 316, 229), ((10000, 4096, 256, 8), 238, 349),
    ((1024, 16384, 512, 1), 351, 1213), ((512, 4096, 512, 1), 96, 248), ((1024, 4096, 384, 1), 95, 216),
    ((8192, 4096, 260, 3), 331, 222), ((10000, 4096, 384, 2), 490, 247), ((16384, 4096, 300, 8), 686, 465),
    ((20000, 2048, 260, 5), 446, 348), ((8192, 4096, 510, 8), 372, 435), ((12300, 16384, 384, 6), 2509, 2850),
    ((33000, 4096, 64, 1), 235, 272), ((70000, 1024, 48, 8), 112, 160),
]


@pytest.mark.parametrize("case,gate,filt", MEASURED, ids=["-".join(map(str, c)) for c, _, _ in MEASURED])
def test_the_faster_gate_is_picked(case, gate, filt):
    assert abs(gate - filt) >= 0.1 * min(gate, filt)
    assert gate_filtered(*case) == (filt < gate)


def test_the_filter_stays_within_its_indexes():
    assert not gate_filtered(1 << 22, 64, 512, 1)  # 2^31 chains at most
    assert not gate_filtered(1 << 22, 16384, 64, 1)


def test_the_gpu_cases_reach_every_gate_kernel():
    from tests.test_gpu_route import GATES
    with open(os.path.join(BLD.CSRC, "gate.hip"), encoding="utf-8") as f:
        src = f.read()
    listed = src[src.index("#define MOE_GATE_CLASSES"):src.index("GateGeometry gate_geometry")]
    kernels = {(int(ec), lm == "true", int(tw)) for ec, lm, tw in re.findall(r"X\((\d+), (true|false), (\d+)\)", listed)}
    assert len(kernels) == 20
    assert {gate_kernel_of(T, E) for T, H, E, k, _ in GATES if not gate_filtered(T, H, E, k)} == kernels
