"""The 32-bit source lists of the hierarchy refresh at their limit: the longest
list that is accepted is walked to its end, and longer ones, whose walk would
wrap around, are refused."""
import ctypes as C
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def sw(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("sw") / "libsw.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "source_walk_check.cpp"),
                    "-o", out], check=True)
    lib = C.CDLL(out)
    lib.sw_fits.argtypes = [C.c_longlong, C.c_longlong]
    lib.sw_pieces.argtypes = [C.c_uint32, C.c_uint32, C.c_int]
    return lib


def test_longest_lists(sw):
    piece = sw.sw_piece()
    longest = 2**32 - piece
    assert sw.sw_fits(longest, longest) and not sw.sw_fits(longest + 1, longest + 1)
    assert sw.sw_fits(7, 2**32) and not sw.sw_fits(7, 2**32 + 1)
    for length in (1, piece - 1, piece, piece + 1, 5 * piece, 5 * piece + 1):
        assert sw.sw_pieces(longest - length, longest, 10) == -(-length // piece)
    # what the limit keeps out: a step past the end that comes out at the front
    assert sw.sw_pieces(2**32 - 1 - piece - 1, 2**32 - 1, 10) == -1
