"""The library's host runtime on the CPU, over stand-ins for the HIP runtime and
the kernels (host_runtime.cpp): what a GPU test cannot see or must not provoke."""
import json
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    d = tmp_path_factory.mktemp("host_runtime")
    inc = ["-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
           "-I" + os.path.join(ROOT, "paper_1904_01567_amd", "csrc")]
    flags = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-D__align__(x)=__attribute__((aligned(x)))",
             "-DHIP_SYMBOL(x)=x", *inc]
    exe = str(d / "host_runtime")
    subprocess.run([*flags, "-x", "c++", os.path.join(ROOT, "paper_1904_01567_amd", "csrc", "gmco_api.hip"),
                    os.path.join(HERE, "host_runtime.cpp"), "-o", exe, "-lpthread"], check=True)

    def run(*args):
        r = subprocess.run([exe, *[str(a) for a in args]], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return json.loads(r.stdout)
    return run


# Results come back whole in whatever pieces they cross, and pinned memory is
# taken once: 24,000 plans of 360 dwells stage 37 MB a call, 200,000 of one dwell
# 74 MB of metrics, 700,000 points 23 MB of case arrays.
@pytest.mark.parametrize("P,K,M", [(1, 1, 40), (24000, 360, 40), (200000, 1, 40), (3, 5, 700000)])
@pytest.mark.parametrize("pinning", [1, 0])
def test_copies_of_any_size(runtime, P, K, M, pinning):
    r = runtime("copies", P, K, M, pinning)
    assert r["ok"] == 1
    assert r["pins"][0] == r["pins"][-1]
    assert r["peak"] <= (64 << 20) + 4096
    assert r["left"] == 0


# Work that a failed call has issued ends before the call returns: its report of
# running plans would otherwise end the next run, here before its first round.
def test_failed_call_leaves_no_report_behind(runtime):
    r = runtime("failed_launch", 14, 18, 40)
    assert r["rc"] == -3
    assert r["pending"] == 0
    assert r["converged"] == 3 and r["work"] == 40
    assert 40 <= r["rounds"] <= 60


# Sampled timing counts the rounds that had running plans and no others: every
# `every`-th of the first `live`, 1 ms an evaluation and 0.1 an update.
@pytest.mark.parametrize("live", [1, 13, 40, 200])
@pytest.mark.parametrize("every", [1, 3, 16])
def test_timing_leaves_empty_rounds_out(runtime, live, every):
    for n, (launches, work, eval_ms, update_ms, rounds) in zip((live, live + 1), runtime("timing", live, every)["runs"]):
        want = -(-n // every)
        assert launches == want and work == want
        assert eval_ms == pytest.approx(want, abs=1e-3) and update_ms == pytest.approx(0.1 * want, abs=1e-3)
        assert rounds >= n


# check_every bounds the rounds between looks at the running plans (8 at most), and
# so those that are issued after the last plan has stopped: a report's distance and
# four more are on their way when the report of no running plan arrives.
@pytest.mark.parametrize("live", [1, 9, 40])
@pytest.mark.parametrize("check_every", [0, 1, 2, 5, 8, 16, 2 ** 31 - 1])
def test_check_every_bounds_the_empty_rounds(runtime, live, check_every):
    r = runtime("checks", live, check_every)
    assert r["converged"] == 3
    period = min(check_every, 8) if check_every else 8
    assert live < r["rounds"] <= live + period + period + 4


# The few-plan forms of the evaluation take a range of 16-point blocks in chunks:
# every block once, in order, up to the largest range that a 32-bit point count has.
def test_few_plan_chunks_cover_every_range(runtime):
    assert runtime("few_chunks")["bad"] == []
