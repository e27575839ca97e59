"""The host driver on the CPU: dpo_host.hip compiled against a stand-in for the
HIP runtime whose kernels do what a check needs (tests/host/checks.cpp)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def checks(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "checks")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-x", "c++", os.path.join(HERE, "host", "checks.cpp"),
                        "-I", os.path.join(HERE, "host"), "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2201_02789_amd", "csrc"), "-pthread", "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


def _run(checks, name):
    r = subprocess.run([checks, name], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, f"{name}: {r.stdout}{r.stderr}"


@pytest.mark.parametrize("name", ["stale_solo", "stale_near", "stale_unposted"])
def test_a_verdict_left_behind_is_nobody_elses(checks, name):
    """A BFS whose launch ticket equals that of a verdict left in the polled
    word waits for its own."""
    _run(checks, name)


def test_a_failed_copy_of_results_reports_no_ticket(checks):
    _run(checks, "failed_copy")


def test_results_for_other_memory_are_copied(checks):
    _run(checks, "foreign_outputs")


@pytest.mark.parametrize("name", ["wide_run", "wide_run_noalloc"])
def test_a_run_of_wide_levels_is_launched_in_growing_parts(checks, name):
    _run(checks, name)


@pytest.mark.parametrize("name", ["batch_symmetric", "batch_directed", "engine_symmetric", "engine_directed"])
def test_bottom_up_nodes_only_where_they_pay(checks, name):
    """A batch's or an engine's replays have them only on arenas found symmetric;
    an engine's only while the running queries are enough work."""
    _run(checks, name)


def test_replays_of_a_batch(checks):
    _run(checks, "batch_replays")
