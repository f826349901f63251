"""What the compiler made of the kernels where a comment in the source says so."""
import re

import pytest

from kernel_code import instructions


@pytest.fixture(scope="module")
def code():
    found = instructions()
    assert len(found) > 500
    return found


def flags(name):
    """What is added to the words per batch of scalar loads in the last template argument of the vector-FMA kernels."""
    m = re.search(r"\d+(?:ihelm_pencil|transform_pencil|convection_pencil|convection_rect)_kernelI\w*?Li(\d+)EEEv", name)
    return int(m.group(1)) & ~255 if m else 0


def test_accesses_keep_their_address_space(code):
    """A FLAT access has no form with a scalar base and is waited for together with LDS and scalar loads."""
    flat = {name: n for name, lines in code.items() if (n := sum(x.startswith("flat_") for x in lines))}
    assert not flat


def test_anisotropic_addresses_are_a_scalar_base_and_a_lane_offset(code):
    kernels = {name: lines for name, lines in code.items() if re.search(r"\d+ihelm_aniso_\w*kernelI", name)}
    assert len(kernels) >= 20
    for name, lines in kernels.items():
        assert not any(x.startswith("v_lshl_add_u64") for x in lines), name
        stores = [x for x in lines if x.startswith("global_store")]
        assert stores and all(re.search(r"s\[\d+:\d+\]", x) for x in stores), name


def test_convection_loads_first_waits_for_no_load_before_the_last_is_out(code):
    """4x4x1 form, last template argument LOADS_FIRST; up to the first barrier."""
    kernels = {name: lines for name, lines in code.items() if re.search(r"\d+convection_mm_kernelI\w*Lb1EEEv", name)}
    assert len(kernels) >= 10
    for name, lines in kernels.items():
        lines = lines[:lines.index("s_barrier")]
        loads = [k for k, x in enumerate(lines) if x.startswith("global_load")]
        waits = [k for k, x in enumerate(lines) if x.startswith("s_waitcnt") and "vmcnt" in x and k > loads[0]]
        assert loads[-1] < waits[0], name


def test_matrices_are_touched_before_one_wait_each(code):
    """Settings with kWarm (256 in the last template argument): one scalar load per 64-byte line and the last word, then a wait."""
    kernels = {name: lines for name, lines in code.items() if flags(name) & 256}
    assert len(kernels) >= 20
    for name, lines in kernels.items():
        sizes = [int(x) for x in re.findall(r"L[ib](\d+)E", name)]
        words = sizes[0] * (sizes[1] if "convection_rect" in name else sizes[0])
        runs, run = [], 0
        for x in lines[:lines.index("s_barrier")]:
            if re.match(r"s_load_dword s\d+,", x):
                run += 1
            elif x.startswith("s_waitcnt") and "lgkmcnt" in x and run:
                runs.append(run)
                run = 0
        matrices = 2 if "convection" in name else 3
        single = -(-words * 8 // 64) + (1 if words % 8 != 1 else -1)       # the last word of an odd matrix comes with the one before
        assert runs == [single] * matrices, name


def test_arguments_are_preloaded_unless_held(code):
    """A kernel with preloaded arguments begins with the branch over the part that loads them where the hardware did not."""
    kernels = {name: lines for name, lines in code.items() if re.search(r"\d+(ihelm|transform)_pencil_kernelI", name)}
    assert len(kernels) > 200
    for name, lines in kernels.items():
        forward = "transform" in name and int(re.findall(r"L[ib](\d+)E", name)[4])
        held = flags(name) & (512 if forward else 1024)
        assert any(x.startswith("s_branch") for x in lines[:8]) == (held == 0), name
    assert 20 <= sum(flags(name) >= 512 for name in kernels) <= 80
