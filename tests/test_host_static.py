"""rotconv_pool_fwd_static accepts a layer only if all that the call touches fits its scratch (host logic only)."""
import os
import subprocess

import pytest

from paper_2512_08888_amd import build as rb

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("static") / "host_static_need")
    libdir = os.path.dirname(rb.LIB)
    flags = [f for f in rb.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", *flags, "-I", os.path.join(rb.ROOT, "include"),
                    "-I", rb.CSRC, os.path.join(HERE, "host_static_need.cpp"), "-o", exe, "-L", libdir, "-l:" + os.path.basename(rb.LIB),
                    "-Wl,-rpath," + libdir], check=True, stderr=subprocess.DEVNULL)
    return exe


@pytest.mark.parametrize("seed", [1, 2])
def test_average_pooling_plans_touch_no_more_than_was_accepted(checker, seed):
    """Random layers of one to four channels and odd rows (their averaged plan runs on padded rows) up to the scratch's size."""
    r = subprocess.run([checker, str(seed)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert "too small 0" in r.stdout and int(r.stdout.split("accepted ")[1].split()[0]) > 500
