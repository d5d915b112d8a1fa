"""The library's host code over a stand-in for the HIP runtime (CPU): host_harness.cpp compiles
mist_host.cpp against it and runs one scenario per test."""

import os
import shutil
import subprocess

import pytest

from paper_2503_19050_amd import mist

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2503_19050_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include/hip"),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("harness") / "host_harness")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__", "-w",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-isystem", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "host_harness.cpp"), os.path.join(CSRC, "mist_plan.cpp"),
                    "-o", exe], check=True)
    return exe


def run(harness, *args):
    r = subprocess.run([harness, *args], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, (r.returncode, (r.stdout + r.stderr)[-2000:])
    return r.stdout


def test_results_are_read_behind_the_null_stream(harness):
    """Every read waits for the evaluation's stream, then runs on the null stream of the space's device
    whichever device is current, and leaves that device current."""
    run(harness, "order_of_reads")


def test_ids_past_the_space_are_refused(harness):
    """Results that no evaluation has written are reported as MIST_E_RANGE, not decoded."""
    run(harness, "ids_out_of_range")


def test_candidate_tiles_are_whole_or_absent(harness):
    """A host allocation that fails while the exact frontier's tiles are cut leaves no partial table."""
    run(harness, "candidate_tiles")


def test_exact_frontier_starts_over_after_a_failure(harness):
    """Every copy, device allocation and host allocation of the first exact frontier fails in turn; the
    next call has whole tables."""
    run(harness, "exact_tables")


def test_which_spaces_are_searched(harness):
    """The sizes from which a space is searched with bounds, by device count and weight samples."""
    run(harness, "search_rule")


def test_running_out_of_memory_is_reported(harness):
    """Calls return MIST_E_NOMEM when every host allocation from some point on fails, their error text's too."""
    run(harness, "out_of_memory")


LAUNCHES = r"""
#include <cstdio>
#include "mist_internal.h"
int main() {
  mist::EvalArgs a{};  // no tile: nothing is launched
  a.R = 5;
  for (int mode = -1; mode < 8; ++mode) std::printf("%d %d\n", mist::launch_eval(a, 1, mode, nullptr), mist::launch_search(a, 1, mode, nullptr));
}
"""


def test_launches_refuse_variants_they_do_not_have(tmp_path):
    """The evaluation kernel has the bucket, weight-sample and dump variants; the search has all six."""
    if not os.path.exists(mist.LIB_PATH):
        pytest.skip("libmist.so is not built")
    (tmp_path / "l.cpp").write_text(LAUNCHES)
    exe = str(tmp_path / "l")
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", CSRC, str(tmp_path / "l.cpp"),
                    mist.LIB_PATH, "-Wl,-rpath," + mist.PKG, "-Wl,--allow-shlib-undefined", "-o", exe], check=True)
    env = dict(os.environ, HIP_VISIBLE_DEVICES="")
    out = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=120, check=True).stdout.split()
    ok = [(int(e) == 0, int(s) == 0) for e, s in zip(out[::2], out[1::2])]
    assert ok == [(m in (0, 1, 3), 0 <= m <= 5) for m in range(-1, 8)]
