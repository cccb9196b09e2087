"""Host code of the plans: the tile list in orbits is the one its definition
gives, and making it costs about what the list in windows costs (it is made on
every call of g4_accumulate_into); a list of rows summed once adds each row
once; the routes of launches to kernels hold over many shapes."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
@pytest.mark.parametrize("driver", ["tile_lists", "kernel_routes", "pair_rows"])
def test_host_driver(tmp_path, driver):
    exe = str(tmp_path / driver)
    src = [os.path.join(ROOT, "tests", "host", driver + ".cpp"),
           os.path.join(ROOT, "tests", "host_sanitize", "launch_stubs.cpp")]
    # host-only translation units, as in the sanitizer build of the same code
    r = subprocess.run(["hipcc", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "include"), *src, "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout
