"""The transposed starlet pass on the host (starlet_host.cpp), with a thread per work item."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2402_08725_amd", "csrc")


@pytest.mark.parametrize("N,J", [(16, 2), (17, 4), (40, 5)])
def test_each_pixel_is_handed_over_once(tmp_path, N, J):
    """By work groups of 256 threads, one per pixel of a tile, and of 512: the functor that
    finishes PSF mode's gradient adds to it and updates the parameters."""
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text("")  # (its names are in starlet_host.cpp)
    exe = str(tmp_path / "starlet_host")
    subprocess.run(["g++", "-std=c++20", "-O1", "-pthread", "-I", str(tmp_path), "-I", CSRC,
                    os.path.join(HERE, "starlet_host.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe, str(N), str(J)], capture_output=True, text=True, check=True, timeout=120).stdout
    assert out.split() == ["256", "1", "1", "512", "1", "1"]
