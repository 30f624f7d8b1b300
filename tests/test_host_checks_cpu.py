"""The library's host code on the CPU (tests/native/host_checks.cpp): HIP calls
on host memory, no GPU."""
import importlib.util
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def host_checks():
    spec = importlib.util.spec_from_file_location("build_native", os.path.join(HERE, "native", "build_native.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    exe = mod.build_host_checks()

    def run(*args):
        r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0 and r.stdout.endswith("ok\n"), (args, r.stdout, r.stderr)
        return r.stdout

    return run


@pytest.mark.parametrize("rows,cols,last", [
    (299_521, 299_521, 2561), (307_201, 307_201, 2817), (299_522, 299_522, 2), (299_523, 299_523, 3), (299_519, 299_519, 7679),
    (299_520, 299_520, 7680), (262_144, 52_993, 4353)])
def test_staged_segments_stay_in_their_buffers(host_checks, rows, cols, last):
    """Staged column segments of numbers of columns that equal parts would leave
    one over (the first two), whose last segment has two columns, three, all
    but one and all, and with columns that no row uses: every index of the
    product inside its buffer, the sums exact."""
    out = host_checks("staged", rows, cols, 33 if cols > 53_000 else 24)
    assert out.startswith("taken") and f"{last} in the last" in out


def test_staged_segments_have_no_single_last_column(host_checks):
    """The width of segments over numbers of columns and widest segments."""
    host_checks("widths")


@pytest.mark.parametrize("rows,cols,per_row", [(262_144, 33_000, 12), (196_608, 16_384, 4), (196_608, 40_000, 20)])
def test_staged_segments_need_one_per_group(host_checks, rows, cols, per_row):
    """Fewer segments than groups: no layout is built."""
    assert "not built" in host_checks("staged", rows, cols, per_row)


def test_products_on_several_streams_are_ordered(host_checks):
    """Products and a solve through one handle on several streams: each that
    shares the staged sums waits for the one before, and nothing is recorded
    or waited for under capture."""
    host_checks("streams")


def test_trainer_stage_after_a_failed_allocation(host_checks):
    """Steps of a trainer, smaller and then larger, after its page-locked
    allocation failed once: none writes past the buffer."""
    host_checks("stage")


def test_mixed_precision_keeps_no_staged_segments(host_checks):
    """Their memory is given back, and float64 builds the same layout again."""
    host_checks("mixed")


def test_abandoned_launch_is_solved_with_separate_kernels(host_checks):
    """A one-launch solve whose workgroups did not all run at once."""
    host_checks("abandoned")
