"""Chunks of a Greeks pass's kept states (state_chunk.hpp), on the host: whole wavefronts,
16 GiB of states or 32,768 paths, a quarter of the free memory at most, and less where an
allocation does not fit, down to one wavefront of 64 paths."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = "/opt/rocm/include"
GIB = 1 << 30


def per_path(n, s):
    return 4 * (s * n * (n + 1) // 2 + n * s + 2 * n)


@pytest.fixture(scope="module")
def chunk(tmp_path_factory):
    if not os.path.isdir(ROCM):
        pytest.skip("HIP headers not available")
    exe = str(tmp_path_factory.mktemp("chunk") / "state_chunk")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I", ROCM,
                    "-I", os.path.join(ROOT, "paper_1006_3340_amd", "csrc"),
                    os.path.join(HERE, "helpers", "state_chunk_driver.cpp"), "-o", exe],
                   check=True, capture_output=True)

    def run(n, s, paths, free=280 * GIB, limit=280 * GIB):
        args = [exe, *map(str, (per_path(n, s), paths, free, limit))]
        out = subprocess.run(args, capture_output=True, text=True, check=True, timeout=20).stdout
        got, requests, ok = map(int, out.split())
        if ok:
            assert got % 64 == 0 and got * per_path(n, s) <= limit
            assert got >= min(64, paths)
        return got if ok else None
    return run


def test_a_pass_that_fits_is_one_chunk(chunk):
    assert chunk(40, 10, 1 << 18) == 1 << 18
    assert chunk(3, 1, 1) == 64
    assert chunk(3, 1, 65) == 128


def test_chunks_are_even(chunk):
    got = chunk(40, 10, 1 << 20)
    parts = -(-(1 << 20) // got)
    assert got * per_path(40, 10) <= 16 * GIB and parts * got - (1 << 20) < 64 * parts


def test_long_periods_still_fill_the_gpu(chunk):
    assert chunk(40, 250, 1 << 17) == 32768
    assert chunk(40, 400, 1 << 17) == 32768


@pytest.mark.parametrize("free", [2 * GIB, 24 * GIB])
def test_a_quarter_of_the_free_memory_at_most(chunk, free):
    assert chunk(40, 10, 1 << 20, free=free) * per_path(40, 10) <= free / 4


@pytest.mark.parametrize("s,limit", [(10, GIB), (300, GIB), (400, GIB // 4), (100_000, 25 * GIB)])
def test_less_where_memory_is_short_down_to_one_wavefront(chunk, s, limit):
    got = chunk(40, s, 1 << 18, limit=limit)
    assert got is not None and (got == 64 or 4 * got * per_path(40, s) > limit)


def test_one_wavefront_is_the_least(chunk):
    assert chunk(40, 400, 1 << 18, limit=64 * per_path(40, 400)) == 64
    assert chunk(40, 400, 1 << 18, limit=64 * per_path(40, 400) - 1) is None
