"""The exchange between the K ranges of a tile where they are not all on the chip together: no range depends on one that does not run."""
import ctypes
import os
import subprocess

import pytest

from paper_2502_08145_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("split") / "split_exchange.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-shared", "-fPIC", "-pthread", "-I" + build.CSRC,
                    os.path.join(HERE, "split_exchange_host.cpp"), "-o", so], check=True)
    fn = ctypes.CDLL(so).split_exchange_run
    fn.argtypes = [ctypes.c_int] * 3 + [ctypes.c_uint32] * 2 + [ctypes.POINTER(ctypes.c_uint32)]
    return fn


@pytest.mark.parametrize("splits", [2, 3, 4, 5, 6, 8])
@pytest.mark.parametrize("slots", [1, 2, 3, 8])
def test_every_share_is_finished_once_with_all_its_sums(run, splits, slots):
    tiles = 5
    flags = (ctypes.c_uint32 * (tiles * splits * (splits - 1)))()
    for epoch, probes in ((1, 0), (1, 0), (1, 2), (0xFFFFFFFE, 1), (0x80000000, 50)):   # the same epoch again: a replayed launch
        moved = run(tiles, splits, slots, epoch, probes, flags)
        if slots == 1:   # one workgroup at a time: the last range of a tile finishes all of them
            assert moved == tiles * (splits - 1)
        else:
            assert 0 <= moved <= tiles * (splits - 1), moved


def test_ranges_that_run_together_finish_their_own(run):
    flags = (ctypes.c_uint32 * (2 * 12))()
    assert run(2, 4, 8, 7, 1 << 30, flags) == 0
