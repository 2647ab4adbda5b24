"""The hand-over's walk with the chunks of the narrower layers: the checks of test_handover_host on the other chunk length."""
import ctypes
import subprocess

import pytest

import test_handover_host as wide


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("handover_narrow")
    src, so = str(d / "model.cpp"), str(d / "model.so")
    with open(src, "w") as f:
        f.write(wide.SOURCE.replace("kSteps", "kStepsNarrow"))
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-unknown-pragmas", "-I" + wide.CSRC, "-o", so, src],
                   check=True)
    return ctypes.CDLL(so)


@pytest.mark.parametrize("T", wide.LENGTHS)
def test_narrow_chunks(lib, T):
    assert lib.steps_per_chunk() == 8
    wide.test_every_chunk_is_walked_whole(lib, T, True)
    wide.test_every_chunk_is_walked_whole(lib, T, False)
    wide.test_a_counted_chunk_has_arrived(lib, T)
