"""The walks' launches on devices of several sizes (a whole one, and partitions
of it with fewer compute units), without a GPU: a program that answers the HIP
calls itself prints what the library would launch. A workgroup's slice, as the
kernel works it out from the launch's own grid, must fit the LDS the launch
gives it, and a request's workgroups must fit on the device together.
"""
import os
import shutil
import subprocess

import pytest

import paper_2609_33652_amd as tsb

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.dirname(tsb.LIB_PATH)


@pytest.fixture(scope="module")
def ref(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not available")
    if not os.path.exists(tsb.LIB_PATH):
        from paper_2609_33652_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("walk") / "ref")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    r = subprocess.run([cxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I" + rocm + "/include", "-rdynamic",
                        os.path.join(HERE, "walk_launch_ref.cpp"), "-o", exe, "-L" + PKG, "-ltsubame",
                        "-Wl,-rpath," + PKG, "-L" + rocm + "/lib", "-lamdhip64", "-Wl,-rpath," + rocm + "/lib"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return exe


# vocabularies of one and several workgroups, of held slices of both widths,
# and of slices that are recomputed
@pytest.mark.parametrize("entry,D", [("rrs", 16), ("traversal", 1), ("traversal", 64)])
@pytest.mark.parametrize("V", [1024, 4097, 50001, 151936, 262208, 303104, 303105, 1212416, 1212420])
@pytest.mark.parametrize("cus", [4, 32, 64, 128, 256])
def test_slice_fits_its_lds(ref, cus, V, entry, D):
    for R in (1, 3, 64):
        r = subprocess.run([ref, str(cus), str(V), str(R), str(D), entry], capture_output=True, text=True)
        assert r.returncode == 0, (r.returncode, r.stdout, r.stderr[-500:])
        G, span, held, lds, need = (int(x) for x in r.stdout.split())
        assert 1 <= G <= cus and G * span >= V, (R, G, span)
        stack = 72 * (D + 1) if entry == "traversal" else 0  # a traversal's stack comes before its slice
        assert lds >= need + stack, (R, G, span, held, lds, need)
        assert lds <= 160 << 10
