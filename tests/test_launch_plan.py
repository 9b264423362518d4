"""The launch plans of the attention and of the projections, without a GPU: they are plain host code,
compiled here by themselves.

Which kernel a call runs follows from its queries, pairs and key tiles alone, or from a projection's rows,
channels and number of matrices.  The GPU tests name the kernels and widths they are for; this file checks
that their sizes still lead there, so that a changed rule cannot quietly leave a kernel without its tests."""
import os
import subprocess

import pytest

import test_gpu_parity as parity
import test_gpu_variants as variants
from paper_2512_02541_amd import build as b

DRIVER = r"""
#include <stdio.h>
#include "agg_attn_plan.h"
int main() {
  long long nq, npairs, tiles;
  while (scanf("%lld %lld %lld", &nq, &npairs, &tiles) == 3) {
    const agg::TilePlan p = agg::plan_tiles(nq, (int)npairs, tiles);
    printf("%d %d %d %d %d %d\n", p.n_full, p.n_tail, p.tail_q, p.tails_last, p.split,
           (int)agg::redo_in_place(tiles));
  }
}
"""


LINEAR_DRIVER = r"""
#include <stdio.h>
#include "agg_linear_plan.h"
int main() {
  long long rows;
  int channels, count;
  while (scanf("%lld %d %d", &rows, &channels, &count) == 3) {
    const agg::LinearPlan p = agg::plan_linear(rows, channels, channels, count, count == 1);
    printf("%lld %d\n", (long long)p.split, p.edge);
  }
}
"""


def _compile(d, text):
    (d / "plan.cpp").write_text(text)
    exe = str(d / "plan")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-Wno-unused-function", "-I", b.CSRC,
                           "-o", exe, str(d / "plan.cpp")])
    return exe


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    """(queries, pairs, keys) -> (kernel width of the last workgroups or "split", redone in place)"""
    exe = _compile(tmp_path_factory.mktemp("plan"), DRIVER)

    def ask(nq, npairs, nkeys):
        text = "%d %d %d\n" % (nq, npairs, -(-nkeys // 64))
        out = subprocess.run([exe], input=text, text=True, check=True, stdout=subprocess.PIPE).stdout
        n_full, n_tail, tail_q, _, split, redo = (int(x) for x in out.split())
        # every query belongs to exactly one workgroup, and none is empty
        last = n_tail if n_tail else n_full
        width = tail_q if n_tail else 256
        assert (n_full + n_tail) * npairs > 0 and (n_full == 0 or n_tail == 0 or tail_q in (128, 192))
        assert n_full * 256 + n_tail * tail_q >= nq > n_full * 256 + n_tail * tail_q - width and last > 0
        return "split" if split else (tail_q if n_tail else 0), bool(redo) and not split

    return ask


def test_every_query_has_a_workgroup(plan):
    for npairs in (1, 7, 16, 20, 255, 256, 300, 5000):
        for nq in (1, 127, 128, 129, 255, 256, 257, 1374, 4096, 10441, 54960):
            for nkeys in (1, 64, 65, 449, 513, 8129):
                plan(nq, npairs, nkeys)


def test_key_sweeps_reach_their_kernels(plan):
    for nkeys in parity.TILE_EDGE_COUNTS:
        # one frame of two heads: shared keys from two tiles on
        assert (plan(nkeys, 2, nkeys)[0] == "split") == (nkeys > 64), nkeys
        redo = nkeys <= 127 * 64
        for width, nq in variants.QUERIES_BY_WIDTH.items():
            assert plan(nq, 16, nkeys) == (width, redo), (nkeys, width)
        assert plan(nkeys, 33 * 8, nkeys)[0] != "split"
        assert plan(nkeys, 33 * 8, nkeys)[1] == redo, nkeys


def test_query_sweeps_reach_their_kernels(plan):
    for nq in variants.QUERY_EDGES:
        assert plan(nq, 9 * 29, (nq + 2) // 3) == (0, True), nq
    for nq, width in variants.QUERY_EDGES_BY_PAIR.items():
        assert plan(nq, 9 * 29, 520) == (width, True), nq


def test_redo_cases_reach_their_kernels(plan):
    routes = set()
    for kind, cases in variants.REDO.items():
        for nq, npairs, nkeys, width in cases:
            got = plan(nq, npairs, nkeys)
            assert got == (width, nkeys <= 127 * 64), (kind, nq, npairs, nkeys, got)
            routes.add((kind, *got))
    # compacted and index-driven: three widths, in place and by the second launch; rows in place likewise
    for kind in ("keys", "list"):
        assert {r for r in routes if r[0] == kind} == {(kind, w, r) for w in (0, 128, 192) for r in (False, True)}
    assert {r[1:] for r in routes if r[0] in ("dense", "frame")} == {(w, r) for w in (0, 128, 192) for r in (False, True)}


def test_tail_cases_reach_their_kernels(plan):
    want = ["split", 192, 192, 192, 192, 192, 192, 0, 192]
    assert [plan(nq, B * H, -(-nq // s))[0] for B, nq, H, s in variants.TAILS] == want
    assert [plan(L, 256, L)[0] for L in (449, 600, 700, 769)] == [0, 128, 192, 128]


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    """[(rows, channels, matrices: three, or one with the residual)] -> [(rows in the first of two launches or 0, edge of the others' tiles)]"""
    exe = _compile(tmp_path_factory.mktemp("linear"), LINEAR_DRIVER)

    def ask(sizes):
        text = "".join("%d %d %d\n" % s for s in sizes)
        out = subprocess.run([exe], input=text, text=True, check=True, stdout=subprocess.PIPE).stdout
        got = [tuple(int(x) for x in line.split()) for line in out.splitlines()]
        assert len(got) == len(sizes)
        return got

    return ask


def _route(split, edge):
    return "256+%d" % edge if split else "%d" % edge


def test_every_row_has_a_tile(tiles):
    sizes = [(rows, 64 * heads, count) for heads in (1, 2, 3, 4, 5, 8, 16, 20, 33, 40, 64) for count in (1, 3)
             for rows in (1, 63, 64, 65, 255, 256, 257, 5496, 10922, 21984, 43521, 65536, 137400, 457542, 1099200)]
    for (rows, channels, count), (split, edge) in zip(sizes, tiles(sizes)):
        assert edge in (64, 128, 256) and 0 <= split < rows and split % 256 == 0
        assert edge != 256 or split == 0
        # tiles of 64: at most two per CU
        few = -(-(rows - split) // 64) * (channels // 64) * count
        assert edge != 64 or few <= 512
        # the rows in a launch of their own fill whole rounds of one large tile per CU, but for less than a token tile
        large = split // 256 * (-(-channels // 256)) * count
        assert split == 0 or large > 0 and -large % 256 < -(-channels // 256) * count


def test_projection_cases_reach_their_kernels(tiles):
    seen = set()
    for cases in (variants.PROJECTIONS, variants.FEW_PROJECTIONS):
        for (heads, rows), want in cases.items():
            got = tiles([(rows, 64 * heads, 3), (rows, 64 * heads, 1)])
            assert tuple(_route(*g) for g in got) == want, (heads, rows, got)
            for residual, (split, edge) in enumerate(got):
                seen.add((edge, residual, heads))
                if split:
                    seen |= {(256, residual, heads), ("behind 256", edge, residual)}
    # with and without the residual: one to five k steps in tiles of 64; one, two, three and five in tiles of
    # 128; three, the fewest that take tiles of 256
    for residual in (0, 1):
        for steps in (1, 2, 3, 5):
            assert (64, residual, steps) in seen and (128, residual, steps) in seen
        assert (64, residual, 4) in seen and (256, residual, 3) in seen
    for (heads, rows), want in variants.SAME_BITS.items():
        got = tiles([(r, 64 * heads, count) for r in (rows, 66) for count in (3, 1)])
        assert tuple(_route(*g) for g in got) == want + ("64", "64"), (heads, rows, got)
    assert {("behind 256", edge, residual) for edge in (64, 128) for residual in (0, 1)} <= seen


# (rows, channels, matrices) -> us by tiles, of a projection among what surrounds it in a block, on one of three boxes
MEASURED = {
    (71776, 64, 1): {"128": 6.359, "256": 10.08, "256+128": 10.4, "256+64": 9.799},
    (29556, 128, 3): {"128": 7.559, "256": 11.8, "256+128": 13.6},
    (59367, 256, 3): {"128": 30.2, "256": 29.8, "256+128": 34.04},
    (29869, 256, 1): {"128": 8.239, "256": 12.96},
    (21960, 320, 3): {"128": 20.92, "256": 31.08, "256+128": 29, "256+64": 26.28},
    (11452, 512, 3): {"128": 20.8, "256": 30.95, "256+128": 26.28, "256+64": 23.52},
    (32968, 512, 1): {"128": 24.36, "256": 36.4, "256+128": 30.08, "256+64": 26.52},
    (56076, 512, 3): {"128": 101.4, "256": 99.55, "256+128": 94.35},
    (7201, 768, 3): {"128": 29.92, "256": 43.44, "256+128": 35.76, "256+64": 30.88},
    (48475, 768, 1): {"128": 83.43, "256": 90.39, "256+128": 83.63},
    (5651, 1024, 3): {"128": 39.04, "256": 52.11, "256+128": 42.4, "256+64": 36.4},
    (5651, 1024, 1): {"128": 16.2, "256": 28.52},
    (11029, 1024, 3): {"128": 73.35, "256": 80.11, "256+128": 69.87, "256+64": 63.83},
    (21960, 1024, 3): {"128": 140.7, "256": 134.5, "256+128": 125.8, "256+64": 119.4},
    (21960, 1024, 1): {"128": 57.15, "256": 64.07, "256+128": 59.59},
    (92600, 1024, 3): {"128": 624.9, "256": 487.8, "256+128": 499.2},
    (13981, 1152, 3): {"128": 119.2, "256": 119.3, "256+128": 108.3},
    (5874, 1280, 3): {"128": 67.99, "256": 66.07, "256+128": 59.19},
    (4284, 1536, 3): {"128": 71.03, "256": 76.15, "256+128": 60.47},
    (6076, 2048, 3): {"128": 162.9, "256": 151.9, "256+128": 139.1},
    (19490, 2048, 1): {"128": 178.2, "256": 178, "256+128": 165.7},
    (2523, 2560, 3): {"128": 116.4, "256": 125.7, "256+128": 97.83},
    (2014, 3072, 3): {"128": 136.8, "256": 145.5, "256+128": 110.7},
    (1480, 4096, 3): {"128": 176.2, "256": 189.5, "256+128": 140.1},
    (4796, 4096, 1): {"128": 188.1, "256": 208.9, "256+128": 156.9},
    (2958, 4096, 3): {"128": 330.9, "256": 300.2, "256+128": 277},
    (20166, 4096, 1): {"128": 792.5, "256": 612.6, "256+128": 639.9},
    (103206, 1024, 1): {"128": 264.2, "256": 240.4, "256+128": 235.5},
}


def test_projections_take_what_was_measured_faster(tiles):
    """Within 6 % of the best choice: between two choices boxes differ by as much."""
    for size, got in zip(MEASURED, tiles(list(MEASURED))):
        took, best = MEASURED[size][_route(*got)], min(MEASURED[size].values())
        assert took <= 1.06 * best, (size, got, took, best)
