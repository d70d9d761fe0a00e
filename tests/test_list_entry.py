"""The list kernel's entry words on the host: csrc/list_entry.h compiled as
plain C++.  An entry is session << 12 | slot and uses every 32-bit value, so
the one of the largest session (2^20 - 1) in the last slot (4,095) equals the
word that stands for none."""
import ctypes
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2609_09643_amd", "csrc")
SRC = """
#include "list_entry.h"
using namespace unison;
extern "C" uint32_t word(uint32_t sid, uint32_t slot) { return list_word(sid, slot); }
extern "C" uint32_t sid(uint32_t w) { return list_sid(w); }
extern "C" uint32_t slot(uint32_t w) { return list_slot(w); }
extern "C" uint32_t rows(uint64_t n) { return list_rows(n); }
extern "C" uint32_t pick(uint32_t hl, uint32_t sl, uint32_t h, uint32_t s) { return fired_in_sram(hl, sl, h, s); }
"""
TOP, LAST, NONE = (1 << 20) - 1, 4095, 0xFFFFFFFF


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("list_entry")
    cpp, so = str(d / "e.cpp"), str(d / "e.so")
    open(cpp, "w").write(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", CSRC, cpp, "-o", so],
                   check=True)
    L = ctypes.CDLL(so)
    for f in (L.word, L.sid, L.slot, L.rows, L.pick):
        f.restype = ctypes.c_uint32
    L.rows.argtypes = [ctypes.c_uint64]
    for f in (L.word, L.sid, L.slot, L.pick):
        f.argtypes = [ctypes.c_uint32] * (4 if f is L.pick else 2 if f is L.word else 1)
    return L


def expire_all(lib, hbm, sram):
    """The kernel's expiry loop over two sets of fired entries: while a list has
    a leaf with a fired entry, the smaller of the lists' smallest words leaves."""
    order = []
    while hbm or sram:
        h, s = min(hbm, default=NONE), min(sram, default=NONE)
        if lib.pick(len(hbm), len(sram), h, s):
            assert s in sram, "picked the SRAM list, where nothing fired"
            sram.remove(s)
            order.append(s)
        else:
            assert h in hbm, "picked the HBM list, where nothing fired"
            hbm.remove(h)
            order.append(h)
    return order


@pytest.mark.parametrize("tier", ["hbm", "sram"])
@pytest.mark.parametrize("others", [0, 1, 5])
def test_the_largest_session_in_the_last_slot_expires(lib, tier, others):
    top = lib.word(TOP, LAST)
    assert (lib.sid(top), lib.slot(top)) == (TOP, LAST)
    rng = random.Random(others)
    for _ in range(50):
        words = {lib.word(rng.randrange(TOP), rng.randrange(4096)) for _ in range(others)}
        hbm = {w for w in words if rng.random() < 0.5}
        sram = words - hbm
        (sram if tier == "sram" else hbm).add(top)
        want = sorted(hbm | sram)
        assert expire_all(lib, hbm, sram) == want


def test_words_round_trip(lib):
    for s in (0, 1, 77, TOP - 1, TOP):
        for t in (0, 1, 63, 64, LAST - 1, LAST):
            w = lib.word(s, t)
            assert (lib.sid(w), lib.slot(w)) == (s, t)
