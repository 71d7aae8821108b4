"""Launch arithmetic that is plain C++ (csrc/*.h without device code), compiled
for the host and checked over whole ranges."""
import ctypes
import heapq
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_13499_amd", "csrc")
CXX = shutil.which("g++") or shutil.which("c++")
CUS = 256

pytestmark = pytest.mark.skipif(CXX is None, reason="no host C++ compiler")


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("launch_shapes")
    src, so = str(d / "launch_shapes.cpp"), str(d / "launch_shapes.so")
    with open(src, "w") as f:
        f.write('''
#include "gemm_schedule.h"
using namespace opscale;
extern "C" {
void chain(int group, int rounds, int chained, int* out) {
  const Chain c = chain_of(group, rounds, chained != 0);
  out[0] = c.first, out[1] = c.len;
}
int64_t grid(int64_t items, int chained, int exact) { return chain_grid(items, chained != 0, exact != 0); }
}
''')
    subprocess.run([CXX, "-std=c++17", "-O1", "-shared", "-fPIC", f"-I{CSRC}", src, "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.grid.restype = ctypes.c_int64
    lib.grid.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int]
    return lib


# ------------------------------------------- chains of the four-wave GEMM ---
def _chains(host, items, grid, chained=1):
    """The item numbers of each workgroup, as the kernel derives them."""
    rounds = -(-items // CUS)
    c, out = (ctypes.c_int * 2)(), []
    for wg in range(grid):
        host.chain(wg // CUS, rounds, chained, c)
        out.append(list(range(c[0] * CUS + wg % CUS, min(items, (c[0] + c[1]) * CUS), CUS)))
    return out


@pytest.mark.parametrize("chained", [0, 1])
def test_chains_cover_every_item_once(host, chained):
    for items in [1, 255, 256, 257, 511, 768, 896, 984, 1024, 1025, 1535, 1536, 1537, 2048, 2900, 3072, 3920, 8624]:
        wgs = _chains(host, items, host.grid(items, chained, 1), chained)
        assert sorted(i for w in wgs for i in w) == list(range(items)), items
        assert all(wgs), "no workgroup without an item"
        # a grid for at most 8624 items serves this number too
        more = _chains(host, items, host.grid(8624, chained, 0), chained)
        assert sorted(i for w in more for i in w) == list(range(items)), items


def test_chain_grid_of_an_upper_bound(host):
    """Any upper bound's grid has the workgroups that fewer items need."""
    need = [0]
    for rounds in range(1, 600):
        need.append(max(need[-1], host.grid(rounds * CUS, 1, 1)))
        assert host.grid(rounds * CUS - 255, 1, 0) >= need[-1], rounds


def _makespan(costs, cus):
    """Workgroups in order, each to the CU that is free first (one per CU)."""
    free, end = [0.0] * cus, 0.0
    for c in costs:
        t = heapq.heappop(free) + c
        end = max(end, t)
        heapq.heappush(free, t)
    return end


@pytest.mark.parametrize("cus", [13, 26, 64, 96, 128, 154, 160, 192, 205, 224, 230, 243, 255, 256])
def test_chains_on_a_share_of_the_cus(host, cus):
    """On any number of CUs a chained launch takes no longer than one item per
    workgroup does, counted in tile times (a split tail's items take a half to
    a quarter of one)."""
    for tiles in list(range(257, 2700, 61)) + [896, 984, 840, 560, 1024, 3920]:
        for split in (1, 2, 3, 4):
            tail = tiles % CUS if split > 1 else 0
            if split > 1 and (tail == 0 or tail * split > CUS):
                continue
            cost = [1.0] * (tiles - tail) + [1.0 / split] * (tail * split)
            wgs = _chains(host, len(cost), host.grid(len(cost), 1, 1))
            chained = _makespan([sum(cost[i] for i in w) for w in wgs], cus)
            assert chained <= _makespan(cost, cus) + 1e-9, (tiles, split)


def test_long_launches_are_chained(host):
    """Most items of a long launch sit in chains (16 rounds: half of them have a
    tile before them)."""
    for items, least in ((3920, 0.5), (8624, 0.6), (2 * 8624, 0.65)):
        wgs = _chains(host, items, host.grid(items, 1, 1))
        assert sum(len(w) - 1 for w in wgs) >= least * items
