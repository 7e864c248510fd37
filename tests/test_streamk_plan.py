"""Host logic of the GEMM planning (csrc/streamk.hpp, csrc/layout.hpp), checked by brute-force C++
programs compiled with the host compiler under the address and undefined-behaviour sanitizers:
  * the balanced K split: every workgroup's segments for a range of (tiles per group, K slabs,
    workgroups per group) give exact single coverage, valid slot numbers and load balance;
  * the tile heights: all rows covered, the plans of measured sizes, and of the sizes that GPU tests were made for;
  * the carving of the `saved` buffer and the two workspaces, and the K partitions the planner
    picks, over a range of shapes and compute-unit counts.
The headers are the ones the kernels and the entry points include."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SAN = ["-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-g", "-O1", "-std=c++17"]


def _run(tmp_path, name, text=None):
    exe = str(tmp_path / name)
    src = os.path.join(ROOT, "tests", "cpp", name + ".cpp")
    subprocess.run(["g++", *SAN, src, "-o", exe], check=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=600, env=env)
    assert r.returncode == 0, r.stdout + r.stderr
    return r


def _build_and_run(tmp_path, name, min_cases):
    r = _run(tmp_path, name)
    assert r.stdout.startswith("ok "), r.stdout + r.stderr
    assert "runtime error" not in r.stderr and "AddressSanitizer" not in r.stderr, r.stderr
    assert int(r.stdout.split()[1]) > min_cases


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_streamk_partition_bruteforce_under_sanitizers(tmp_path):
    _build_and_run(tmp_path, "streamk_check", 10000)


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_buffer_carving_and_k_partitions_under_sanitizers(tmp_path):
    _build_and_run(tmp_path, "layout_check", 500)


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_the_tiles_that_gpu_tests_are_made_for(tmp_path):
    """A changed cost must not empty the GPU tests of tile heights: what their sizes are planned to, by name of the test."""
    from helpers import TWO_PART_GATE_UP
    want = {k: (v, None) for k, v in TWO_PART_GATE_UP.items()}
    # test_gate_up_tile_heights
    for R, inference, training in [(257, "0+4", "0+4"), (385, "0+5", "0+6"), (481, "0+6", "0+6"), (577, "0+7", "3+0"),
                                   (673, "3+0", "3+0"), (769, "0+4", "0+4")]:
        want[R, 264, 8264, False] = (inference, None)
        want[R, 264, 8264, True] = (training, None)
    want[1400, 264, 12808, False], want[1400, 264, 12808, True] = ("0+7", None), ("6+0", None)
    # test_down_tile_heights
    for R, C, I, down in [(257, 1032, 8264, "s8:0+4"), (769, 1032, 8264, "s8:0+5"), (961, 1032, 8264, "s8:0+6"),
                          (1153, 1032, 8264, "s8:0+7"), (1793, 4104, 72, "s1:0+4"), (1921, 4104, 72, "s1:0+5"),
                          (2401, 4104, 72, "s1:0+6"), (2881, 4104, 72, "s1:0+7")]:
        want[R, C, I, False] = (None, down)
    # test_last_tile_row_of_at_most_128_rows
    for R, gate_up in [(257, "0+4"), (300, "0+4"), (384, "0+4"), (385, "0+6"), (513, "0+6"), (640, "3+0"), (868, "0+4")]:
        want[R, 520, 8264, True] = (gate_up, None)
    text = "".join(f"{R} {C} {I} {int(saved)}\n" for R, C, I, saved in want)
    lines = _run(tmp_path, "plan_print", text).stdout.split("\n")
    for (key, plans), line in zip(want.items(), lines):
        for plan, got in zip(plans, line.split(" ")):
            assert plan is None or plan == got, (key, line)
