"""CPU checks of the word that a search's host looks at between rounds (csrc/host_word.h, plain host code): compiled here with g++."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "host_word.h"
static HostWord numbers;
extern "C" uint32_t next() { return numbers.next(); }
extern "C" int arrives(const uint32_t *word) { return numbers.arrives(word); }
extern "C" void pass_over(uint32_t n) { while (n--) numbers.next(); }
"""


@pytest.fixture()
def lib(tmp_path):
    (tmp_path / "word.cpp").write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2506_08276_amd", "csrc"),
                           "-o", str(tmp_path / "word.so"), str(tmp_path / "word.cpp")])
    lib = ctypes.CDLL(str(tmp_path / "word.so"))
    lib.next.restype = ctypes.c_uint32
    lib.pass_over.argtypes = [ctypes.c_uint32]
    return lib


def test_what_an_abandoned_call_stores_is_not_taken_for_a_later_launch_s(lib):
    """A call ends with an error while its kernels run, the next call launches its first: whatever number of the first call's comes
    in late, the wait goes on until the second call's own is there."""
    word = ctypes.c_uint32(0)
    first = [lib.next() for _ in range(3)]
    own = lib.next()
    for late in first:
        word.value = late
        assert not lib.arrives(ctypes.byref(word)), late
    word.value = own
    assert lib.arrives(ctypes.byref(word))


def test_numbers_go_on_past_32_bits(lib):
    lib.pass_over(2**32 - 3)
    word = ctypes.c_uint32(2**32 - 3)
    for _ in range(6):
        last, number = word.value, lib.next()
        assert number != last and not lib.arrives(ctypes.byref(word))
        word.value = number
        assert lib.arrives(ctypes.byref(word))
