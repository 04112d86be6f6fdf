"""CPU tests of the tile tables with one sanitizer each: tests/host_wide_check.cpp checks the tables of rows of
more than four elements (ownership, neighbours, local indices element by element, bounds, the sample the launch
shapes are chosen by) under AddressSanitizer and UBSan; under ThreadSanitizer it and tests/host_chain_check.cpp
run operators that are large enough for tables and row orders on several threads."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2209_00806_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _build(tmp, source, sanitizer):
    cxx = shutil.which("g++")
    if not cxx or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("g++ or the HIP headers are not available")
    out = str(tmp / f"{source}_{sanitizer.split(',')[0]}")
    cmd = [cxx, "-O1", "-g", "-std=c++17", f"-fsanitize={sanitizer}", "-fno-omit-frame-pointer", "-D__HIP_PLATFORM_AMD__",
           "-I/opt/rocm/include", os.path.join(ROOT, "tests", source + ".cpp"),
           os.path.join(ROOT, "paper_2209_00806_amd", "csrc", "host.cpp"), "-pthread", "-o", out]
    subprocess.run(cmd, check=True, capture_output=True, timeout=600)
    return out


@pytest.fixture(scope="module")
def wide_address(tmp_path_factory):
    return _build(tmp_path_factory.mktemp("host_wide"), "host_wide_check", "address,undefined")


@pytest.fixture(scope="module")
def wide_thread(tmp_path_factory):
    return _build(tmp_path_factory.mktemp("host_wide"), "host_wide_check", "thread")


@pytest.fixture(scope="module")
def chain_thread(tmp_path_factory):
    return _build(tmp_path_factory.mktemp("host_wide"), "host_chain_check", "thread")


def _band(n, hops, seed=0, drop=0.0):
    """Rows joined to those at the given distances; drop: share of the bonds left out (rows of uneven length)."""
    rng = np.random.default_rng(seed)
    i = np.repeat(np.arange(n), len(hops))
    j = (i + np.tile(np.asarray(hops), n)) % n
    keep = rng.uniform(size=i.size) >= drop
    return inputs.from_bonds(n, i[keep], j[keep], np.ones(int(keep.sum())), np.zeros(n))


def _files(tmp_path, members):
    rp, cols, inst = [0], [], [0]
    for lat in members:
        cols.append(lat.col.astype(np.int32) + inst[-1])
        rp.extend((lat.row_ptr[1:] + rp[-1]).tolist())
        inst.append(inst[-1] + lat.n_orb)
    paths = [str(tmp_path / n) for n in ("rp", "col", "inst")]
    np.asarray(rp, np.int64).tofile(paths[0])
    np.concatenate(cols).astype(np.int32).tofile(paths[1])
    np.asarray(inst, np.int64).tofile(paths[2])
    return paths


def _run(exe, paths, *args):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1", UBSAN_OPTIONS="halt_on_error=1", TSAN_OPTIONS="halt_on_error=1")
    r = subprocess.run([exe, *paths, *map(str, args)], capture_output=True, text=True, timeout=300, env=env)
    assert r.returncode in (0, 3), (args, r.stdout, r.stderr)
    assert r.stdout.startswith("OK" if r.returncode == 0 else "NOFIT"), (args, r.stdout, r.stderr)
    return r.returncode == 0


CASES = {
    "six": lambda: [_band(700, (1, 2, 50))],
    "uneven_rows": lambda: [_band(900, (1, 2, 3, 31), 1, 0.3)],
    "bilayer": lambda: [inputs.twisted_bilayer(20, 20)],
    "batch": lambda: [_band(33, (1, 3, 5)), _band(401, (1, 2, 17, 40)), _band(64, (1, 2, 3))],
    "full": lambda: [_band(1500, (1, 2, 3, 4, 5, 6, 7, 8, 30, 31, 32, 33), 2)],
}


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("case", sorted(CASES))
def test_wide_tables(wide_address, tmp_path, case, order):
    members = CASES[case]()
    paths = _files(tmp_path, members)
    w = max(int(np.diff(lat.row_ptr).max()) for lat in members)
    fits = 0
    for T, rows in ((256, 4096), (64, 512), (256, 300), (16, 64), (1, 30)):
        for width in {(w + 1) // 2 * 2, 24}:
            fits += _run(wide_address, paths, order, T, width, T, rows)
    assert fits > 0


def test_wide_tables_on_threads(wide_thread, tmp_path):
    """288000 elements and more: tables on two threads or more, the bisection on four."""
    paths = _files(tmp_path, [_band(9000, tuple(range(1, 13))), _band(7000, tuple(range(1, 13)), 3, 0.2)])
    for order in (0, 1):
        assert _run(wide_thread, paths, order, 256, 24, 256, 4096)


def test_chain_tables_on_threads(chain_thread, tmp_path):
    """60000 rows of three elements, seven hops: tables on several threads, tiles halved on each."""
    paths = _files(tmp_path, [inputs.graphene(200, 100), inputs.graphene(90, 50)])
    assert _run(chain_thread, paths, 1, 512, 7, 1024, 1280)
    assert _run(chain_thread, paths, 0, 64, 7, 400, 500)
