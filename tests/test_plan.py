"""The rules that lay work out over the chip (csrc/plan.h), evaluated on the CPU."""
import ctypes
import os
import subprocess

import pytest

from paper_2605_05802_amd.build import CSRC

SOURCE = """
#include "plan.h"
extern "C" {
void shared_tiles(int n_sets, int per_set, int *set, int *part) {
    for (int wg = 0; wg < n_sets * per_set; ++wg) sr::shared_tiles_of(wg, n_sets, per_set, set + wg, part + wg);
}
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, str(d / "plan.cpp"), "-o", str(d / "plan.so")])
    return ctypes.CDLL(str(d / "plan.so"))


@pytest.mark.parametrize("per_set", [1, 2, 3, 7, 313])
@pytest.mark.parametrize("n_sets", [1, 2, 4, 7, 8, 9, 12, 16, 37])
def test_shared_query_tiles_use_every_xcd(plan, n_sets, per_set):
    """Every (set, part) has one workgroup, whole rounds of eight sets stay on one XCD each, and no XCD (workgroup index
    modulo 8) has more than a workgroup above its share: one group's two kv heads used to leave six XCDs idle."""
    n = n_sets * per_set
    s, p = (ctypes.c_int * n)(), (ctypes.c_int * n)()
    plan.shared_tiles(n_sets, per_set, s, p)
    assert sorted(zip(s, p)) == [(a, b) for a in range(n_sets) for b in range(per_set)]
    load = [0] * 8
    home = {}
    for wg in range(n):
        load[wg % 8] += 1
        if s[wg] < n_sets // 8 * 8:
            assert home.setdefault(s[wg], wg % 8) == wg % 8
    assert max(load) <= -(-n // 8)
