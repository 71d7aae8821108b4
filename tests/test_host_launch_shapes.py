"""Launch arithmetic that is plain C++ (csrc/*.h without device code), compiled
for the host and checked over whole ranges."""
import ctypes
import heapq
import os
import shutil
import subprocess

import numpy as np
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
#include "attn_f32_plan.h"
#include "gemm_schedule.h"
#include "grid.h"
using namespace opscale;
extern "C" {
void attn_f32(int64_t B, int64_t T, int64_t longest, int64_t Hq, int64_t D, int64_t* out) {
  const AttnF32Plan p = attn_f32_plan(B, T, longest, Hq, D);
  out[0] = p.row_len, out[1] = p.items, out[2] = p.levels, out[3] = p.grid;
}
// first row, rows and workgroups of each launch; the number of launches
int rows(int64_t M, int per_wg, int64_t* out, int most) {
  int n = 0;
  launch_rows(M, per_wg, [&](int64_t m, int64_t r, uint32_t grid) {
    out[3 * n] = m, out[3 * n + 1] = r, out[3 * n + 2] = grid;
    return ++n == most ? 1 : 0;
  });
  return n;
}
int rms_wave(int64_t M, int64_t H, int64_t nvec, int cus) { return rmsnorm_wave_rows(M, H, nvec, cus); }
int add_wave(int64_t M, int64_t H, int cus) { return add_rmsnorm_wave_rows(M, H, cus); }
double moe_tiles(int64_t rows, int64_t N, int64_t E) { return grouped_tiles(rows, N, E); }
int moe_deep(int64_t rows, int64_t N, int64_t E, int cus) { return grouped_deep_ring(rows, N, E, cus); }
int waves(int64_t N, int splits, int cus) { return stream_waves(N, splits, cus); }
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
    lib.attn_f32.argtypes = [ctypes.c_int64] * 5 + [ctypes.c_void_p]
    lib.attn_f32.restype = None
    lib.rows.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_void_p, ctypes.c_int]
    lib.rms_wave.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int]
    lib.add_wave.argtypes = [ctypes.c_int64] * 2 + [ctypes.c_int]
    lib.moe_tiles.argtypes = [ctypes.c_int64] * 3
    lib.moe_tiles.restype = ctypes.c_double
    lib.moe_deep.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int]
    lib.waves.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int]
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


# ------------------------------------- rings of the MoE decode-batch GEMM ---
def test_grouped_tile_estimate(host):
    """The estimate against evenly routed lists."""
    rng = np.random.default_rng(5)
    for rows, N, E in ((4, 5376, 16), (32, 6144, 16), (56, 5760, 32), (2048, 5120, 64), (512, 4096, 8), (2, 28672, 8),
                       (256, 16384, 4), (4096, 3584, 64), (1, 512, 1)):
        tiles = np.mean([(-(-np.bincount(rng.integers(0, E, rows), minlength=E) // 64)).sum() for _ in range(400)])
        assert host.moe_tiles(rows, N, E) == pytest.approx(tiles * -(-N // 256), rel=0.06), (rows, N, E)


def test_grouped_ring_rule(host):
    """The deep ring where the launch's last round of 512 tiles holds at most 256
    (E experts of one column block a tile each; every expert gets a row)."""
    for E, deep in ((1, 1), (84, 1), (250, 1), (262, 0), (336, 0), (500, 0), (520, 1), (760, 1), (780, 0), (1020, 0)):
        assert host.moe_deep(20 * E, 256, E, CUS) == deep, E
    # exactly 256 past a whole round (1280 tiles): every one of 64 experts has rows
    assert host.moe_deep(2048, 5120, 64, CUS) and not host.moe_deep(2048, 3584, 64, CUS)
    assert not any(host.moe_deep(20 * E, 256, E, CUS - 1) for E in range(1, 600, 7)), "a share of the CUs: never"


# ------------------------------------------- the decode-batch linear's waves ---
@pytest.mark.parametrize("cus", [8, 13, 26, 64, 128, 154, 192, 205, 230, 243, 255])
def test_stream_waves_on_a_share_of_the_cus(host, cus):
    """On no share does another workgroup shape give a CU fewer columns, the
    workgroups dealt evenly to the 32 shader engines."""
    even = cus if cus < 32 else cus // 32 * 32
    for N in list(range(8, 3000, 56)) + list(range(3000, 60000, 488)) + [4096, 6144, 10240, 28672, 57344]:
        for splits in (1, 2, 3, 4, 8):
            wgs = lambda w: -(-N // (16 * w)) * splits
            cost = lambda w: -(-wgs(w) // even) * w
            assert cost(host.waves(N, splits, cus)) == min(cost(w) for w in (5, 6, 7, 8)), (N, splits)
    # gate-up and QKV of the 8B layer: whole passes
    for share, gate_up, qkv in ((255, 8, 7), (230, 8, 7), (205, 5, 8), (192, 5, 8), (154, 7, 6), (128, 7, 6)):
        assert (host.waves(28672, 1, share), host.waves(6144, 4, share)) == (gate_up, qkv), share


# ------------------------------------------------- fp32 prefill attention ---
def _attn(host, B, T, longest, Hq, D):
    out = (ctypes.c_int64 * 4)()
    host.attn_f32(B, T, longest, Hq, D, out)
    return list(out)


@pytest.mark.parametrize("D", [64, 128])
def test_attn_f32_plan(host, D):
    """Whatever the batch and however loose the bound: a launch that HIP takes,
    with an item for every tile and not many more, or a wave per token where
    that is one launch for all."""
    rng = np.random.default_rng(D)
    cases = [(1024, 1024 * 16, 16384, 32), (128, 131072, 131072, 32), (2048, 2047 * 4 + 8192, 8192, 32),
             (1, 1 << 26, 1 << 30, 8), (1, 1 << 30, 1 << 30, 1), (1 << 24, 1 << 24, 1, 4), (3000, 3000, 2**31 - 1, 64),
             (1, 128, 128, 4), (256, 7680, 30, 4), (64, 64, 4096, 4), (1, 1, 1, 1)]
    for _ in range(3000):
        B = int(2 ** rng.uniform(0, 12))
        T = int(B * 2 ** rng.uniform(-2, 12)) + 1
        cases.append((B, T, min(2**31 - 1, int(-(-T // B) * 2 ** rng.uniform(0, 14))), int(2 ** rng.uniform(0, 7))))
    for B, T, longest, Hq in cases:
        row_len, items, levels, grid = _attn(host, B, T, longest, Hq, D)
        if items == 0:
            assert row_len == 2**31 - 1 and T * 64 < 2**32
            continue
        assert 1 <= grid <= items and grid * 256 < 2**32, (B, T, longest, Hq)
        assert row_len == 0 or T * 64 < 2**32
        # at most 2.25 times the tiles that B prompts of T tokens can have, heads each
        assert items <= 2.25 * (T // 32 + B) * Hq, (B, T, longest, Hq)
        if levels:
            assert row_len == 0 and items == B * levels * Hq and levels * 32 >= min(longest, T)
        else:  # any split of T into B prompts: L // 32 + 1 tiles a prompt of more than row_len tokens
            assert items >= (T // 32 + min(B, T // (row_len + 1))) * Hq


# -------------------------------------------------------- one row a group ---
@pytest.mark.parametrize("per_wg", [1, 4])
def test_rows_past_one_grid(host, per_wg):
    """Rows past what one grid holds go into further launches, each row once."""
    most = (2**24 - 1) * per_wg
    for M in (1, 2, 5, 2**24 - 1, 2**24, 2**24 + 5, most - 1, most, most + 1, 2 * most, 2 * most + 3, 2**31 - 1):
        out = (ctypes.c_int64 * 3072)()
        n = host.rows(M, per_wg, out, 1024)
        at = 0
        for i in range(n):
            m, r, grid = out[3 * i:3 * i + 3]
            assert m == at and r > 0 and grid * 256 < 2**32 and (grid - 1) * per_wg < r <= grid * per_wg, (M, i)
            at += r
        assert at == M
    # an error ends it
    assert host.rows(3 * most, per_wg, (ctypes.c_int64 * 9)(), 2) == 2


def test_norm_rows_on_a_share_of_the_cus(host):
    """A wave a row only on a share, for row blocks that fill it, and for rows
    that a wave holds: any others keep their workgroup, up to the most rows."""
    for H, vec in ((1032, 8), (4096, 8), (8192, 8), (516, 4), (4096, 4)):
        for cus in (8, 26, 64, 128, 154, 160):
            rms, add = -(-20480 * cus // H), -(-40960 * cus // H)
            assert host.rms_wave(rms, H, H // vec, cus) and not host.rms_wave(rms - 1, H, H // vec, cus)
            assert host.add_wave(add, H, cus) == (H <= 4096) and not host.add_wave(add - 1, H, cus)
            assert host.rms_wave(2**31 - 1, H, H // vec, cus)
        for cus in (161, 192, 255, CUS):
            assert not host.rms_wave(2**31 - 1, H, H // vec, cus) and not host.add_wave(2**31 - 1, H, cus)
    assert not host.rms_wave(8871, 8200, 1025, 64) and not host.rms_wave(8871, 4100, 1025, 64)
    assert not host.add_wave(8871, 4104, 64)
