"""The policy that keeps device blocks between calls, on the CPU: which block a
call takes, which have to go, and that returning one allocates nothing (it
happens in destructors).  Blocks are numbers, streams and devices too."""
import ctypes as C
import os
import subprocess
import threading

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MB, GB = 1 << 20, 1 << 30
BUDGET = 64 * GB
KEEP_BLOCKS, KEEP_CALLS = 16, 32


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("blocks") / "libblocks.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wl,-Bsymbolic",
                    "-I" + os.path.join(ROOT, "paper_1410_1629_amd", "csrc"),
                    os.path.join(ROOT, "tests", "helpers", "blocks_emu.cpp"), "-o", so], check=True)
    lib = C.CDLL(so)
    u64, i32 = C.c_ulonglong, C.c_int
    for name, args, res in (("blocks_reset", [], None), ("blocks_news", [], u64), ("blocks_set_over", [i32, i32], None), ("blocks_call", [], None),
                            ("blocks_keep", [i32, u64, i32, i32], i32), ("blocks_take", [u64, i32, i32], i32),
                            ("blocks_excess", [i32, u64], i32), ("blocks_drop", [i32], i32),
                            ("blocks_idle_bytes", [i32], u64), ("blocks_budget", [u64, u64], u64)):
        getattr(lib, name).argtypes, getattr(lib, name).restype = args, res
    return lib


@pytest.fixture
def S(lib):
    lib.blocks_reset()
    return lib


def _gone(S, dev, budget=BUDGET):
    out = []
    while True:
        q = S.blocks_excess(dev, budget)
        if not q:
            return out
        out.append(q)


def test_a_call_takes_the_smallest_block_that_fits(S):
    for q, size in ((1, 300 * MB), (2, 100 * MB), (3, 2 * GB)):
        assert S.blocks_keep(q, size, 0, 7)
    assert S.blocks_take(3 * GB, 0, 7) == 0
    assert S.blocks_take(90 * MB, 0, 7) == 2
    assert S.blocks_take(90 * MB, 0, 7) == 1
    assert S.blocks_take(90 * MB, 0, 7) == 0  # the last one is more than four times as large
    assert S.blocks_take(90 * MB, 1, 7) == 0 and S.blocks_take(600 * MB, 0, 7) == 3


def test_a_block_in_use_on_another_stream_is_left(S):
    S.blocks_keep(1, 100 * MB, 0, 7)
    S.blocks_set_over(1, 0)
    assert S.blocks_take(90 * MB, 0, 8) == 0
    assert S.blocks_take(90 * MB, 0, 7) == 1  # its own stream waits for it by order


def test_the_per_thread_stream_is_another_in_each_thread(S):
    """Its handle (2) is the same everywhere; calls of two threads on it must not wait for one another."""
    S.blocks_keep(1, 100 * MB, 0, 2)
    S.blocks_set_over(1, 0)
    got = []
    t = threading.Thread(target=lambda: got.append(S.blocks_take(90 * MB, 0, 2)))
    t.start()
    t.join()
    assert got == [0]
    assert S.blocks_take(90 * MB, 0, 2) == 1


def test_the_budget_takes_the_longest_unused(S):
    for q in range(1, 5):
        S.blocks_keep(q, 10 * GB, 0, 7)
        S.blocks_call()
    assert _gone(S, 0) == []
    assert _gone(S, 0, 25 * GB) == [1, 2]
    assert S.blocks_idle_bytes(0) == 20 * GB and S.blocks_idle_bytes(1) == 0
    assert _gone(S, 0, 0) == [3, 4]


def test_what_a_device_may_keep(S):
    assert S.blocks_budget(200 * GB, 288 * GB) == 64 * GB  # 64 GiB
    assert S.blocks_budget(60 * GB, 64 * GB) == 16 * GB    # or a quarter of the device
    assert S.blocks_budget(144 * GB, 288 * GB) == 64 * GB
    assert S.blocks_budget(144 * GB - 1, 288 * GB) == 0    # nothing with less than half of it free


def test_a_device_keeps_so_many_blocks(S):
    for q in range(1, KEEP_BLOCKS + 4):
        S.blocks_keep(q, MB, 0, 7)
        S.blocks_call()
    assert _gone(S, 0) == [1, 2, 3]


def test_a_block_goes_when_calls_do_not_use_it(S):
    """Age counts calls, not the blocks they ask for (a run with a peel-ray queue asks for two)."""
    S.blocks_keep(1, MB, 0, 7)
    for _ in range(KEEP_CALLS):
        S.blocks_call()
        for _ in range(3):
            S.blocks_take(1 << 50, 0, 7)
        assert _gone(S, 0) == []
    S.blocks_call()
    S.blocks_keep(2, MB, 0, 7)
    assert _gone(S, 0) == [1]


def test_a_device_that_is_no_longer_used_gives_its_blocks_back(S):
    """Calls on one device let the blocks of another grow old too; one whose last use goes on is left for later."""
    S.blocks_keep(1, GB, 0, 7)
    S.blocks_keep(2, GB, 0, 7)
    S.blocks_set_over(2, 0)
    for _ in range(KEEP_CALLS):
        S.blocks_call()
    S.blocks_keep(3, GB, 1, 8)
    assert _gone(S, 1) == []
    S.blocks_call()
    S.blocks_keep(4, GB, 1, 8)
    assert _gone(S, 1) == [1]
    S.blocks_set_over(2, 1)
    assert _gone(S, 1) == [2] and S.blocks_idle_bytes(1) == 2 * GB


def test_each_device_has_blocks_of_its_own(S):
    """A device that holds its full number of idle blocks leaves the others theirs."""
    for q in range(1, KEEP_BLOCKS + 1):
        S.blocks_keep(q, MB, 0, 7)
    S.blocks_keep(100, 10 * MB, 1, 8)
    assert _gone(S, 1) == [] and _gone(S, 0) == []
    assert S.blocks_take(10 * MB, 1, 8) == 100


def test_drop_empties_a_device_or_all(S):
    for q, dev in ((1, 0), (2, 1), (3, 0), (4, 2)):
        S.blocks_keep(q, MB, dev, 7)
    assert sorted([S.blocks_drop(0), S.blocks_drop(0)]) == [1, 3] and S.blocks_drop(0) == 0
    assert sorted([S.blocks_drop(-1), S.blocks_drop(-1)]) == [2, 4] and S.blocks_drop(-1) == 0


def test_nothing_allocates(S):
    """Blocks are returned from destructors, which must not throw, however many there are."""
    kept = 0
    for q in range(1, 4000):
        kept += S.blocks_keep(q, MB, q % 8, 7)
    assert kept >= 8 * KEEP_BLOCKS
    for _ in range(kept):
        assert S.blocks_drop(-1)
    assert S.blocks_drop(-1) == 0 and S.blocks_news() == 0
