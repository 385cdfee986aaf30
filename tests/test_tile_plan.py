"""The tile arithmetic of the prefill GEMMs (csrc/tile_plan.h), built with g++ and run on
the host: an expert's token rows are covered once by its tiles whatever their number."""
import ctypes
import os
import shutil
import subprocess

import pytest

import _tile_plan as copy

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_16473_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")):
        pytest.skip("needs g++ and the HIP headers")
    so = str(tmp_path_factory.mktemp("tile_plan") / "libtile_plan.so")
    cmd = [cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-fsanitize=undefined", "-fsanitize-undefined-trap-on-error",
           "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"), "-I", CSRC,
           os.path.join(ROOT, "tests", "native", "tile_plan.cpp"), "-o", so]
    build = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert build.returncode == 0, build.stderr[-4000:]
    return ctypes.CDLL(so)


def test_tiles_cover_every_row(lib):
    # every small count, then counts whose blocks times tiles pass 32 bits (the first is
    # 5,931,521) up to the largest pair count that an int holds with its rounding
    big = [5931520, 5931521, 6000000, 8388608, 16777215, 16777217, 100000001, 2 ** 31 - 1 - 256]
    for c in list(range(1, 5000)) + big:
        assert lib.check_rows(c) == 0, c


@pytest.mark.parametrize("slots", [1, 32])
def test_plans_cover_every_tile(lib, slots):
    out = (ctypes.c_int * 4)()
    for U in (1, 7, 8, 9, 31, 255, 256, 257, 1000, 4099):
        for nsteps in (2, 7, 8, 64, 224):
            for planes, maxparts in ((1, 0), (1, 64), (4, 0), (4, 23), (8, 0)):
                at = 0
                for xcd in range(8):
                    lib.plan(U, nsteps, slots, planes, maxparts, 100, xcd, out)
                    u0, units, full, s = out
                    assert u0 == at and units >= 0 and full <= units
                    r = units - full
                    assert (s == 1 and r == 0) or (1 < s <= 16 and 0 < r < slots and full % slots == 0)
                    assert s <= min(planes, 4) or r * s <= (slots if s <= planes else maxparts)
                    assert s == 1 or nsteps // s >= 4
                    assert all(lib.xcd_of(U, u) == xcd for u in range(u0, u0 + units))
                    at += units
                assert at == U


def test_operand_offsets(lib):
    # f is bounded by memory alone: one slab of d = 128, f = 8.5 million is 6.5 GB, and the 256
    # rows of a down tile then span more than 32 bits
    lib.offset_of.restype = ctypes.c_size_t
    for K in (128, 14336, 8421376, 8500096, 33554432, 306783488, 2 ** 31 - 128):
        for row, at in ((0, 0), (7, 112), (64, 0), (252, 96), (255, 112), (2 ** 31 - 1, 112)):
            assert lib.offset_of(row, K, at) == 2 * row * K + at


@pytest.mark.parametrize("d,f,experts,T", [(128, 14336, 1, 1), (384, 14336, 1, 1), (384, 14336, 1, 127),
                                           (640, 8192, 2, 1), (1408, 5632, 2, 1), (1408, 5632, 2, 15)])
def test_short_prompts_fill_the_down_projection(lib, d, f, experts, T):
    # few tiles: at least as many work groups as four K parts of 128-row tiles would give
    out = (ctypes.c_int * 4)()
    groups = 0
    for xcd in range(8):
        lib.plan(experts * ((d + 255) // 256), f // 64, 32, lib.planes_of(T), 0, T * experts, xcd, out)
        groups += out[2] + (out[1] - out[2]) * out[3]
    assert groups >= 4 * experts * (d // 128)


def test_copy_of_the_plan_agrees(lib):
    """tests/_tile_plan.py, which the GPU tests pick their shapes with."""
    out = (ctypes.c_int * 4)()
    assert all(copy.max_planes(T) == lib.planes_of(T) for T in range(1, 600))
    for U in (0, 1, 8, 31, 97, 256, 272, 1000):
        for nsteps in (2, 9, 24, 88, 224):
            for slots, planes, maxparts, pairs in ((32, 1, 0, 5), (32, 1, 64, 900), (32, 4, 24, 900), (32, 8, 0, 5),
                                                   (32, 8, 48, 250), (31, 4, 64, 64)):
                for xcd, p in enumerate(copy.plan(U, nsteps, slots, planes, maxparts, pairs)):
                    lib.plan(U, nsteps, slots, planes, maxparts, pairs, xcd, out)
                    assert tuple(out) == p, (U, nsteps, slots, planes, maxparts, pairs, xcd)
