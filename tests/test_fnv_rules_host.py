"""The rules that choose between one lane per item and many (CPU only): at
shapes where both sides were timed on MI355X the rule takes the faster one."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1705_06965_amd", "csrc")
CUS = 256

WRAPPER = """
#include "fnv_rules.hpp"
extern "C" int group_rule(uint64_t n, uint32_t item, uint32_t wg, uint32_t cus) {
  return gsys_k::many_lanes(n, item, wg, gsys_k::helped_block(wg, gsys_k::ceil_div(n, wg), cus));
}
extern "C" int consume_rule(uint64_t n, uint32_t item) { return gsys_k::consume_many_lanes(n, item); }
extern "C" int consume_grid_rule(uint64_t n, uint32_t item, uint32_t wg, uint32_t grid, uint32_t cus) {
  return gsys_k::consume_many_lanes(n, item, wg, grid, cus);
}
extern "C" int spread_rule(uint64_t n, uint32_t item, uint32_t wg, uint32_t cus, uint64_t slots) {
  return gsys_k::spread_group(n, item, wg, cus, slots);
}
extern "C" int item_rule(uint64_t n, uint32_t item, uint32_t wg) {
  return gsys_k::many_lanes(n, item, wg, wg);
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ is missing")
    d = tmp_path_factory.mktemp("rules")
    (d / "w.cpp").write_text(WRAPPER)
    so = str(d / "librules.so")
    b = subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                        "-I" + CSRC, str(d / "w.cpp"), "-o", so], capture_output=True, text=True)
    assert b.returncode == 0, b.stderr
    lib = C.CDLL(so)
    lib.group_rule.argtypes = [C.c_uint64, C.c_uint32, C.c_uint32, C.c_uint32]
    lib.consume_rule.argtypes = [C.c_uint64, C.c_uint32]
    lib.consume_grid_rule.argtypes = [C.c_uint64] + [C.c_uint32] * 4
    lib.spread_rule.argtypes = [C.c_uint64, C.c_uint32, C.c_uint32, C.c_uint32, C.c_uint64]
    lib.item_rule.argtypes = [C.c_uint64, C.c_uint32, C.c_uint32]
    return lib


# (items, bytes, work-group): chains ahead / many lanes ahead
CHAINS = [(1024, 16448, 1024), (4099, 16448, 1024), (1024, 65600, 1024), (96, 1 << 20, 1024),
          (512, 8256, 512), (2051, 8256, 512), (512, 16448, 512), (2051, 16448, 512),
          (96, 1 << 20, 512), (256, 8256, 256), (1027, 8256, 256), (256, 16448, 256),
          (20000, 512, 64), (8000, 4096, 1024)]
MANY = [(64, 4096, 64), (64, 576, 64), (5003, 4096, 64), (1500, 65536, 64), (64, 1 << 20, 64),
        (128, 4096, 128), (128, 65600, 128), (96, 1 << 20, 256), (12192, 8256, 512),
        (20000, 4096, 512), (6120, 16448, 512), (12192, 8256, 256), (6120, 16448, 256)]


@pytest.mark.parametrize("n,item,wg", CHAINS)
def test_group_calls_take_the_chains(rules, n, item, wg):
    assert not rules.group_rule(n, item, wg, CUS)


@pytest.mark.parametrize("n,item,wg", MANY)
def test_group_calls_take_many_lanes(rules, n, item, wg):
    assert rules.group_rule(n, item, wg, CUS)


@pytest.mark.parametrize("n,wg,many", [(20000, 128, 0), (60000, 256, 0), (60000, 512, 1),
                                       (200000, 1024, 0)])
def test_work_item_calls_that_fill_the_chip(rules, n, wg, many):
    """4 KiB work-item calls, more than 64 per work-group: no helpers, and the
    chains unless those would read the link in 128-byte pieces."""
    assert rules.item_rule(n, 4096, wg) == many


@pytest.mark.parametrize("n,item,wg,slots,want", [
    (64, 4096, 64, 65536, 16), (8000, 4096, 1024, 65536, 32), (60000, 576, 1024, 65536, 256),
    (65536, 576, 1024, 65536, 256), (65537, 576, 1024, 65536, 1024),
    (100000, 576, 1024, 65536, 1024), (100000, 576, 1024, 1 << 18, 512), (5000, 4096, 1024, 4096, 1024),
    (20, 1 << 20, 64, 64, 8), (300, 256, 64, 65536, 64)])
def test_spread_keeps_to_launches_that_fit_the_ring(rules, n, item, wg, slots, want):
    assert rules.spread_rule(n, item, wg, CUS, slots) == want


@pytest.mark.parametrize("n,item,many", [
    (50000, 4096, 1), (200000, 4096, 1), (60000, 8192, 1), (200, 1 << 20, 1), (200000, 640, 0),
    (200000, 1024, 1), (65536, 8256, 0), (33000, 8256, 0), (20000, 8256, 1), (65536, 12288, 0),
    (40000, 16448, 1), (40000, 24576, 1), (5000, 65600, 1), (200000, 512, 0)])
def test_consume_counts_the_last_step(rules, n, item, many):
    assert rules.consume_rule(n, item) == many


@pytest.mark.parametrize("n,item,wg,grid,many", [
    (20000, 4096, 256, 79, 0), (20000, 4096, 64, 313, 0), (20000, 4096, 512, 40, 0),
    (20000, 4096, 1024, 5, 0), (20000, 4096, 1024, 20, 1), (20000, 4096, 1024, 64, 1),
    (20000, 4096, 1024, 256, 1), (20000, 8256, 256, 79, 0), (4000, 65536, 1024, 64, 1),
    (300, 65536, 256, 64, 1), (300, 65536, 256, 2, 1), (20000, 4096, 256, 200, 1),
    (1000, 4096, 256, 64, 1), (20000, 4096, 256, 512, 1), (100, 512, 64, 2, 0)])
def test_consume_with_a_grid(rules, n, item, wg, grid, many):
    assert rules.consume_grid_rule(n, item, wg, grid, CUS) == many
