"""CPU checks of the LDS plan of the search kernel (csrc/advance_plan.h, plain host code): compiled here with g++."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CU_LDS = 160 * 1024
SOURCE = """
#include "advance_plan.h"
extern "C" int fixed_bytes() { return ADV_FIXED; }
extern "C" int plan(int m_sub, int ef, int queries, int pieces, int *near, int *blocks)
{
    const AdvancePlan p = plan_advance(m_sub, ef, queries, 256, pieces);
    *near = p.near;
    *blocks = p.blocks;
    return p.bytes;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2506_08276_amd", "csrc"),
                           "-o", str(d / "plan.so"), str(d / "plan.cpp")])
    return ctypes.CDLL(str(d / "plan.so"))


def plan(lib, m_sub, ef, queries, pieces):
    near, blocks = ctypes.c_int(), ctypes.c_int()
    return lib.plan(m_sub, ef, queries, pieces, ctypes.byref(near), ctypes.byref(blocks)), near.value, blocks.value


def without_rows(m_sub, ef):
    """The table, the queue's keys, CSR rows and marks (read in steps of 256), 64 empty columns at an odd pitch."""
    return m_sub * 1024 + 16 * ef + -(-ef // 256) * 256 + 64 * 8


def on_a_cu(lib, dynamic):
    """Blocks that LDS lets a CU hold; it is handed out in pieces of 1280 bytes."""
    return CU_LDS // (-(-(dynamic + lib.fixed_bytes()) // 1280) * 1280)


def test_every_accepted_search_fits_a_compute_unit(lib):
    """Up to 128 subspaces (what the encoders' widths leave) and queues of up to 1024 entries, with the kernel's fixed arrays."""
    for m_sub in range(1, 129):
        for ef in range(1, 1025):
            for queries, pieces in ((1, 12), (600, 6), (4096, 2)):
                total, near, _ = plan(lib, m_sub, ef, queries, pieces)
                assert total + lib.fixed_bytes() <= CU_LDS and 0 <= near <= 64, (m_sub, ef, queries)
                assert total >= without_rows(m_sub, ef) + (64 * 8 * (near | 1) - 64 * 8), (m_sub, ef, queries)


@pytest.mark.parametrize("pieces", [2, 6, 12, 16])
def test_as_many_queries_share_a_cu_as_the_table_lets(lib, pieces):
    """256 CUs: rows of the approximate queue never keep a query away that table, exact queue and registers leave room for."""
    by_registers = 4 if pieces <= 6 else 3
    for m_sub in (1, 8, 16, 24, 32, 48, 64, 96, 128):
        for ef in (1, 64, 200, 256, 257, 500, 1000, 1024):
            for queries in (1, 272, 273, 528, 529, 832, 833, 1088, 1089, 4096):
                room = min(by_registers, on_a_cu(lib, without_rows(m_sub, ef)))
                total, near, blocks = plan(lib, m_sub, ef, queries, pieces)
                want = min(room, 1 + (queries > 256 + 16) + (queries > 512 + 16) + (queries > 768 + 64))
                assert on_a_cu(lib, total) >= want == blocks, (m_sub, ef, queries)
                # and what is left is used: another two rows would not leave room for them
                assert near == 64 or on_a_cu(lib, total + 2 * 64 * 8) < want or want == 1 and total + 3 * 64 * 8 + lib.fixed_bytes() > CU_LDS
    assert on_a_cu(lib, plan(lib, 16, 200, 1000, 6)[0]) == 4 and on_a_cu(lib, plan(lib, 32, 200, 750, 12)[0]) == 3
