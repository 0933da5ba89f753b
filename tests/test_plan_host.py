"""The library's host side on a stand-in for the HIP runtime (tests/host/plan_check.cpp):
which calls it makes, what it allocates and what it returns where memory is short.
No GPU is used; kernels are not run."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    from paper_2003_13218_amd import binding
    if not shutil.which("g++") or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"):
        pytest.skip("no host compiler or HIP headers")
    if not os.path.exists(binding.LIB_PATH):
        from paper_2003_13218_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("plan") / "plan_check")
    lib = os.path.dirname(binding.LIB_PATH)
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                        os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "host", "plan_check.cpp"), "-o", exe,
                        "-rdynamic", "-L", lib, "-l:libfmm.so", f"-Wl,-rpath,{lib}", "-Wl,--allow-shlib-undefined"],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]

    def run(*args):
        r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=300)
        return r.returncode, r.stdout.strip()
    return run


def test_batch_symmetric_pass_is_not_a_graph_of_old_workspaces(check):
    assert check("batch_replay") == (0, "ok")


def test_new_plan_serves_the_call_that_may_not_allocate(check):
    assert check("plan_then_noalloc") == (0, "ok")


def test_calls_after_one_without_memory(check):
    assert check("call_after_no_memory") == (0, "ok")


def test_workspaces_take_the_memory_of_operators(check):
    assert check("short_of_memory") == (0, "ok")


def test_list_operators_take_the_memory_of_operators(check):
    assert check("lists_short_of_memory") == (0, "ok")


def test_options_report_operators_that_do_not_fit(check):
    assert check("options_without_memory") == (0, "ok")


def test_crowded_leaves_fill_the_chip(check):
    assert check("crowded_leaves") == (0, "ok")


def test_cache_lines_of_other_kernels_are_not_taken(check, tmp_path):
    assert check("old_cache_line", tmp_path / "autotune.txt") == (0, "ok")


def test_batch_waits_for_its_boxes_after_the_last(check):
    assert check("batch_joins") == (0, "ok")


def test_near_field_forks_where_the_far_field_needs_it(check):
    assert check("near_field_fork") == (0, "ok")
