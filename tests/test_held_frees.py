"""Buffers a setup lets go are released only after a wait that covers their use,
also while another thread closes a handle (no GPU needed)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def library():
    from paper_2002_04958_amd import _lib
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2002_04958_amd import build
        build.build(verbose=False)
    return _lib.LIB_PATH


def test_releases_follow_the_wait_that_covers_them(library, tmp_path):
    exe = str(tmp_path / "held_frees")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include",
                    f"-I{ROOT}/include", f"-I{ROOT}/paper_2002_04958_amd/csrc",
                    os.path.join(HERE, "held_frees.cpp"), library, f"-L{ROCM}/lib",
                    "-lamdhip64", f"-Wl,-rpath,{ROCM}/lib",
                    f"-Wl,-rpath,{os.path.dirname(library)}", "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "ok" in r.stdout, (r.returncode, r.stdout, r.stderr)
