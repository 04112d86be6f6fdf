"""CPU checks of the launch decisions of the library's host side:
tests/host_engine_check.cpp, compiled with AddressSanitizer and UBSan (what runs
on several threads with ThreadSanitizer too) against every host source of the
library and a device made of host memory (tests/fake_device.h), whose free
memory a check may change at any time."""
import concurrent.futures as cf
import glob
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ENV = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0", UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1",
           TSAN_OPTIONS="halt_on_error=1")


def _build(tmp_path_factory, sanitizer):
    cxx = shutil.which("g++")
    if not cxx or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("g++ or the HIP headers are not available")
    tmp = str(tmp_path_factory.mktemp("host_engine"))
    srcs = sorted(glob.glob(os.path.join(ROOT, "paper_2209_00806_amd", "csrc", "*.cpp")))
    srcs.append(os.path.join(ROOT, "tests", "host_engine_check.cpp"))
    flags = ["-O1", "-g", "-std=c++17", f"-fsanitize={sanitizer}", "-fno-omit-frame-pointer",
             "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include"]
    objs = [os.path.join(tmp, os.path.basename(s) + ".o") for s in srcs]

    def compile_one(k):
        subprocess.run([cxx, *flags, "-c", srcs[k], "-o", objs[k]], check=True, capture_output=True, timeout=600)

    with cf.ThreadPoolExecutor(max_workers=6) as ex:
        list(ex.map(compile_one, range(len(srcs))))
    out = os.path.join(tmp, "host_engine_check")
    subprocess.run([cxx, *flags, *objs, "-pthread", "-o", out], check=True, capture_output=True, timeout=600)
    return out


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    return _build(tmp_path_factory, "address,undefined")


@pytest.fixture(scope="module")
def thread_checker(tmp_path_factory):
    return _build(tmp_path_factory, "thread")


def _run(exe, name):
    r = subprocess.run([exe, name], capture_output=True, text=True, timeout=300, env=ENV)
    assert r.returncode == 0 and r.stdout.endswith("OK\n"), r.stdout + r.stderr


def test_quasi_eigenstate_runs_share_a_layout(checker):
    """Both runs of a quasi-eigenstate call add to the same accumulators: their states lie in one layout, also
    when the memory that is free changes between the two decisions."""
    _run(checker, "quasi_layout")


def test_bench_pass_after_other_calls(checker):
    """Timing launches follow the last propagation's shape and precision, whatever other calls on the handle
    have made of its tile tables since."""
    _run(checker, "bench_pass")


def test_haydock_step_reads_inside_its_lds(checker):
    """The second product of the Haydock step runs on whole waves; the lanes that have no own row stay inside the
    vector of the evaluated rows."""
    _run(checker, "haydock_places")


def test_tables_are_kept_between_kinds_of_calls(checker):
    """Calls of several kinds in turn on one handle build their tile tables once."""
    _run(checker, "tables_kept")


def test_refused_tile_sizes_are_remembered(checker):
    """A tile size that an operator's rows do not fit is not tried again by every call."""
    _run(checker, "sizes_refused")


def test_irregular_operators_keep_one_order_per_launch(checker):
    """The shapes on tiles with shells are taken where they are the faster ones, by a sample of the tiles."""
    _run(checker, "overlap")


def test_wide_pass_orders_its_tiles_by_size(checker):
    """The order of the wide pass's tiles follows the size of a vector, whatever order is configured."""
    _run(checker, "wide_order")


def test_calls_without_room_for_tables_go_on(checker):
    """Without free memory for the tables of the chain or the wide pass, every method goes on with another shape
    and keeps none of them."""
    _run(checker, "no_room")


def test_room_asked_for_is_what_a_run_takes(checker):
    """The guard before a propagation on tiles counts what the run then allocates, to 1 MiB."""
    _run(checker, "room_is_what_it_takes")


def test_kept_states_are_given_back(checker):
    """Large states of several time steps do not stay on a handle after the call that kept them."""
    _run(checker, "states_given_back")


def test_calls_without_host_memory_for_tables_go_on(checker):
    """Where the host cannot allocate the tile tables, a call goes on with another shape."""
    _run(checker, "no_host_memory")


def test_tiles_of_scattered_rows_are_halved_as_far_as_it_takes(checker):
    """A few tiles of rows that lie apart do not keep an operator from the chain."""
    _run(checker, "scattered_tiles")


def test_hopeless_operators_are_ruled_out_early(checker):
    """A first call on an operator whose balls grow too fast for any tile makes no order and no samples."""
    _run(checker, "ruled_out")


def test_members_are_ordered_on_threads(checker, thread_checker):
    """The row orders of a batch's members, made on several threads, are those each member gets alone."""
    _run(checker, "batch_orders")
    _run(thread_checker, "batch_orders")


def test_tables_on_threads(thread_checker):
    """Tile tables of the chain, made on several threads for calls of several kinds."""
    _run(thread_checker, "tables_kept")
