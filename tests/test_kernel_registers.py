"""Registers of built kernels where a wavefront per SIMD hangs on them (512 vector registers per SIMD lane,
handed out in eights; none of these spills)."""
import re

import pytest

from kernel_metadata import kernels


@pytest.fixture(scope="module")
def built():
    return kernels()


def registers(built, pattern):
    found = [k for name, k in built.items() if re.search(pattern, name)]
    assert found, pattern
    for k in found:
        assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0
    # accumulation registers come out of the same 512
    return [(k[".vgpr_count"] + 7) // 8 * 8 for k in found]


@pytest.mark.parametrize("n,waves", [(7, 8), (8, 8), (9, 8), (10, 5), (11, 4), (12, 4), (13, 4), (14, 4)])
def test_convection_f64(built, n, waves):
    """Without all loads first, units per workgroup as on small batches."""
    g = {9: 3}.get(n, 1)
    split = int(n > 9)
    xcd = int(g % 3 != 0)
    pattern = f"convection_pencil_kernelIdLi{n}ELi{g}ELi2ELb{xcd}ELb{split}ELb0E"
    assert all(512 // r >= waves for r in registers(built, pattern))
