"""The rules by which a call of the 16-bit scans takes one of their instances (csrc/mdn_scan_rules.h), compiled for the host."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_05838_amd", "csrc")
WRAPPERS = """
#include "mdn_scan_rules.h"
extern "C" {
unsigned long long bytes(unsigned long long blocks, int d, bool vt, bool states) { return mdn::scan_bytes(blocks, d, vt, states); }
bool touch(unsigned long long bytes, bool reverse) { return mdn::touch_pays(bytes, reverse); }
bool q_tile(int columns, int d, unsigned long long pairs, unsigned long long chunks, unsigned long long bytes, bool vt, bool states) {
    return mdn::q_tile_pays(columns, d, pairs, chunks, bytes, vt, states);
}
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("rules")
    (tmp / "rules.cpp").write_text(WRAPPERS)
    so = str(tmp / "rules.so")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, "-o", so, str(tmp / "rules.cpp")], check=True)
    lib = ctypes.CDLL(so)
    lib.bytes.restype = ctypes.c_ulonglong
    lib.bytes.argtypes = [ctypes.c_ulonglong, ctypes.c_int, ctypes.c_bool, ctypes.c_bool]
    lib.touch.restype = ctypes.c_bool
    lib.touch.argtypes = [ctypes.c_ulonglong, ctypes.c_bool]
    lib.q_tile.restype = ctypes.c_bool
    lib.q_tile.argtypes = [ctypes.c_int, ctypes.c_int] + 3 * [ctypes.c_ulonglong] + 2 * [ctypes.c_bool]
    return lib


@pytest.mark.parametrize("d", [64, 128])
def test_a_scan_is_weighed_by_its_own_tensors(rules, d):
    """Every tensor that a scan reads or writes once and no other: the reverse scan writes adjoints of the states, but no V~."""
    rows, square, coef, states = 64 * d * 2, 64 * 64 * 2, 64 * 8 * 4, 2 * d * d * 2
    plain = 3 * rows + 2 * square + coef + rows  # k, q, v; T, Bm; coefficients; o
    for blocks in (1, 777, 1 << 25):
        assert rules.bytes(blocks, d, False, False) == blocks * plain
        assert rules.bytes(blocks, d, True, False) == blocks * (plain + rows)
        assert rules.bytes(blocks, d, True, True) == blocks * (plain + rows + states)
        assert rules.bytes(blocks, d, False, True) == blocks * (plain + states)  # dO for v, dv for o


def test_lines_of_the_touch(rules):
    """Sizes (tokens x heads / 64) that forward and backward together, or the forward alone, were faster at on the side taken."""
    for blocks, d, kept, pays in ((20000 // 4, 128, True, True), (8192 // 4, 128, True, False), (26624 // 4, 128, False, True),
                                  (65536 // 4, 64, False, True), (16384 // 4, 64, True, False)):
        assert rules.touch(rules.bytes(blocks, d, kept, kept), False) is pays, (blocks, d, kept)
    for blocks, d, pays in ((8192 // 4, 128, False), (16384 // 4, 128, True), (16384 // 4, 64, False), (28672 // 4, 64, True)):
        assert rules.touch(rules.bytes(blocks, d, False, True), True) is pays, (blocks, d)


# B, tokens, heads, d, columns, what is kept, whether the tile was faster
@pytest.mark.parametrize("B,T,H,d,columns,kept,tile", [
    (4, 2048, 16, 128, 32, "states", True), (4, 2500, 16, 128, 32, "states", True), (4, 4096, 16, 128, 32, "", False),
    (4, 4096, 24, 64, 32, "states", False), (1, 64, 16, 128, 16, "", True), (1, 512, 16, 128, 16, "", True), (1, 777, 16, 128, 16, "", False),
    (1, 4096, 8, 128, 16, "", False), (1, 16384, 4, 128, 16, "", False), (1, 22000, 16, 128, 16, "", True), (1, 4096, 16, 128, 16, "states", True),
    (1, 30000, 4, 128, 16, "vt", False), (1, 30000, 6, 128, 16, "vt", True), (1, 8192, 16, 64, 16, "vt", True), (1, 4096, 8, 64, 16, "", True),
    (1, 4096, 2, 64, 16, "", False), (1, 512, 2, 64, 16, "", True)])
def test_q_tile_where_it_was_faster(rules, B, T, H, d, columns, kept, tile):
    chunks = (T + 63) // 64
    n = rules.bytes(B * H * chunks, d, kept != "", kept == "states")
    assert rules.q_tile(columns, d, B * H, chunks, n, kept != "", kept == "states") is tile
