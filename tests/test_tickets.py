"""Tickets of the workgroups that share a unit: whatever 32 bits are read, the rows they stand for lie in the kept list."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "ccd_ticket.h"
extern "C" int first_row(unsigned ticket, int chunks, int chunk_rows, int k) {
  return ccd::chunk_first_row(ticket, chunks, chunk_rows, k);
}
"""


@pytest.fixture(scope="module")
def first_row(tmp_path_factory):
    d = tmp_path_factory.mktemp("ticket")
    (d / "t.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2410_01518_amd", "csrc"), str(d / "t.cpp"),
                    "-o", str(d / "t.so")], check=True)
    f = ctypes.CDLL(str(d / "t.so")).first_row
    f.argtypes, f.restype = [ctypes.c_uint, ctypes.c_int, ctypes.c_int, ctypes.c_int], ctypes.c_int
    return f


@pytest.mark.parametrize("k,chunk_rows", [(1, 64), (63, 64), (64, 64), (65, 64), (700, 32), (20001, 512), (32768, 128)])
def test_any_ticket_stays_in_the_list(first_row, k, chunk_rows):
    chunks = -(-k // chunk_rows)
    assert [first_row(t, chunks, chunk_rows, k) for t in range(chunks)] == list(range(0, k, chunk_rows))
    # no chunk of this call: just past the last one, signs, products that wrap to zero or to a row of the list
    for t in (chunks, chunks + 1, 0x7FFFFFFF, 0x80000000, 0xFFFFFFFF, 0xFFFFFFFF - chunks, (1 << 32) // chunk_rows,
              (1 << 32) // chunk_rows + 1, (1 << 31) // chunk_rows, 0x3F800000, 0xBF800000):
        assert first_row(t, chunks, chunk_rows, k) == k, hex(t)
