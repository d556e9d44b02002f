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
extern "C" int plan(int m_sub, int ef, int *near)
{
    const AdvancePlan p = plan_advance(m_sub, ef);
    *near = p.near;
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


def plan(lib, m_sub, ef):
    near = ctypes.c_int()
    return lib.plan(m_sub, ef, ctypes.byref(near)), near.value


def test_every_accepted_search_fits_a_compute_unit(lib):
    """Up to 128 subspaces (what the encoders' widths leave) and queues of up to 1024 entries, with the kernel's fixed arrays."""
    for m_sub in range(1, 129):
        for ef in range(1, 1025):
            total, near = plan(lib, m_sub, ef)
            assert total + lib.fixed_bytes() <= CU_LDS and 0 <= near <= 64, (m_sub, ef)
            # the table, the queue's keys, CSR rows and marks (read in steps of 256), 64 columns at an odd pitch
            assert total >= m_sub * 1024 + 16 * ef + -(-ef // 256) * 256 + 64 * 8 * (near | 1), (m_sub, ef)
