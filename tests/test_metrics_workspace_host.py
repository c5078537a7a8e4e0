"""The metrics' workspaces with a HIP runtime whose allocations fail
(tests/host_metrics_driver.cpp): host code only, no GPU."""
import os
import shutil
import subprocess

import pytest

from paper_2203_14906_amd import build, hodmas


@pytest.mark.skipif(shutil.which(build.HIPCC) is None, reason="needs hipcc")
def test_a_failed_pinned_allocation_ends_with_its_call(tmp_path):
    """Where the kept results cannot be allocated a call brings its own: the error
    of the first allocation is not taken for one of the call's launches.  Where that
    fails too the call is out of memory, and the next one works."""
    here = os.path.dirname(os.path.abspath(__file__))
    flags = ["-std=c++17", "-O1", "-I" + os.path.join(build.ROOT, "include")]
    obj, exe = str(tmp_path / "metrics.o"), str(tmp_path / "driver")
    subprocess.run([build.HIPCC] + flags + ["--offload-arch=" + build.ARCH, "--offload-host-only", "-c",
                                            os.path.join(build.CSRC, "hodmas_metrics.hip"), "-o", obj], check=True)
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(build.HIPCC)))
    subprocess.run(["g++", "-no-pie"] + flags + ["-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(rocm, "include"),
                    os.path.join(here, "host_metrics_driver.cpp"), obj,
                    "-Wl,--unresolved-symbols=ignore-all", "-o", exe], check=True)
    for failures, want in ((0, hodmas.OK), (1, hodmas.OK), (2, hodmas.ENOMEM)):
        res = subprocess.run([exe, str(failures), str(want)], capture_output=True, text=True, timeout=60)
        assert res.returncode == 0, (failures, res.stdout, res.stderr)
