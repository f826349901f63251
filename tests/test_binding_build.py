"""What the build does where the native binding cannot be built: the C libraries stand without it."""
import sys

import pytest

from paper_2604_19906_amd import build


@pytest.fixture
def small(tmp_path, monkeypatch):
    """A build of two sources of one line in a folder of its own, with a binding left from an earlier build."""
    src = tmp_path / "csrc"
    src.mkdir()
    (src / "one.cpp").write_text('extern "C" int one() { return 1; }\n')
    (src / "bench_two.cpp").write_text('extern "C" int two() { return 2; }\n')
    for name, value in {"CSRC": src, "OBJ": tmp_path / "obj", "LIB": tmp_path / "lib.so", "BENCH_LIB": tmp_path / "bench.so",
                        "TORCH_BINDING": tmp_path / "_tpo_torch.so"}.items():
        monkeypatch.setattr(build, name, str(value))
    (tmp_path / "_tpo_torch.so").write_bytes(b"left over")
    return tmp_path


def check(folder):
    with pytest.warns(UserWarning, match="not built"):
        build.build(verbose=False)
    assert (folder / "lib.so").exists() and (folder / "bench.so").exists()
    assert not (folder / "_tpo_torch.so").exists()          # it was built from other sources


def test_libraries_without_torch(small, monkeypatch):
    monkeypatch.setitem(sys.modules, "torch", None)
    check(small)


def test_libraries_without_a_compiler_for_the_binding(small):
    (small / "csrc" / "torch_binding.cpp").write_text("#error\n")
    check(small)
