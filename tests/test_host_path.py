"""The host side of the actor step, run on a HIP runtime that launches nothing (tests/c/host_path.cpp): no GPU is used."""
import os
import subprocess

import pytest

from paper_2605_16154_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def host_path(tmp_path_factory):
    if not os.path.exists(build.LIB):
        build.build_library()
    exe = str(tmp_path_factory.mktemp("host_path") / "host_path")
    cmd = [build._hipcc(), "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-I",
           os.path.join(ROOT, "include"), "-I", build.CSRC, os.path.join(ROOT, "tests", "c", "host_path.cpp"), "-o", exe, "-L", build.PKG,
           "-l:libpcm.so", "-Wl,-rpath," + build.PKG]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def _run(exe, what):
    r = subprocess.run([exe, what], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:] + r.stderr[-1000:]


def test_every_product_stays_inside_the_buffers_of_the_call(host_path):
    """Operands, results and partial products of every launch lie inside what the caller gave, the workspace being as long as
    its query says: over narrow and wide heads (up to a million columns, where a sum of parts no longer fits the buffer of the
    small ones), short and long batches, row panels, and every option."""
    _run(host_path, "bounds")


def test_a_launch_that_fails_is_reported(host_path):
    """Each launch of a call fails in turn, in the stub runtime: the call returns PCM_EHIP, whichever launch it was."""
    _run(host_path, "errors")


def test_fp32_calls_accept_the_workspace_of_the_direct_route(host_path):
    """An fp32 call takes the least workspace that any call of its shape takes, whatever its options: nothing reaches beyond it."""
    _run(host_path, "least")
