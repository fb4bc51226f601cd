"""The tests' model of the 16-bit GEMM launcher's tile choice (helpers.gemm_plan, helpers.head_plan) against the launcher's own
code: the cost tables and plan_tiles are cut out of the source, compiled for the host and asked about the same launches.  The GPU
tests assert through the model which tile a shape takes, so a retuned table cannot empty them unnoticed."""
import ctypes
import importlib.util
import itertools
import os
import subprocess

import pytest

from tests import helpers as H

GLUE = """
#include <algorithm>
#include <cstdint>
static constexpr int BK = 64;
static int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }
%s
extern "C" void plan(int heads, int M, int ncols, int K, int glu, int *out) {
  const TilePlan p = heads ? plan_tiles(kHeadCost, kHeadKinds, M, ncols, K, glu) : plan_tiles(kTileCost, kTileKinds, M, ncols, K, glu);
  out[0] = p.rows_big;
  out[1] = p.kind;
}
"""


@pytest.fixture(scope="module")
def launcher(tmp_path_factory):
    src = open(H.GEMM_SOURCE).read()
    text = src[src.index("struct TileCost {"):src.index("template <typename OT, int EPI>\nstatic int launch_kind(")]
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(GLUE % text)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-o", str(d / "plan.so"), str(d / "plan.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "plan.so"))

    def ask(heads, M, ncols, K, glu=False):
        kinds = [t[0] for t in (H._tile_table(src, "kHead256", "kHeadCost") if heads else H._tile_table(src, "kTile256", "kTileCost"))]
        out = (ctypes.c_int * 2)()
        lib.plan(int(heads), M, ncols, K, int(glu), out)
        big, kind = out[0], kinds[out[1]]
        return [(big, kinds[0]), (M - big, kind)] if big else [(M, kind)]
    return ask


ROWS = [1, 5, 31, 33, 64, 65, 100, 129, 200, 300, 391, 513, 777, 1154, 1500, 2000, 2600, 2707, 2900, 3500, 4100, 5000, 7168, 9001, 12001, 16384, 20001]


def test_gemm_plan_is_the_launchers(launcher):
    seen = set()
    for M, N, K, glu in itertools.product(ROWS, (40, 512, 1000, 2096, 4104, 6144, 24576), (64, 192, 320, 704, 1024, 2560, 4096, 12288), (False, True)):
        got = H.gemm_plan(M, N, K, glu)
        assert got == launcher(False, M, N // 2 if glu else N, K, glu), (M, N, K, glu)
        seen |= {k for _, k in got} | ({"split"} if len(got) == 2 else set())
    assert len(seen) == 9                                    # every tile and the split occur


def test_head_plan_is_the_launchers(launcher):
    seen = set()
    for M, (nq, nkv), K in itertools.product(ROWS, ((2, 1), (4, 2), (8, 8), (16, 8), (24, 8), (32, 8)), (64, 256, 1024, 2560, 4096)):
        got = H.head_plan(M, nq, nkv, K)
        assert got == launcher(True, M, (nq + 2 * nkv) * 128, K), (M, nq, nkv, K)
        seen |= {k for _, k in got} | ({"split"} if len(got) == 2 else set())
    assert len(seen) == 5
    assert all(k != "kHead256" for M in ROWS for _, k in H.head_plan(M, 3, 3, 1024))        # an odd number of heads


@pytest.fixture(scope="module")
def loops():
    spec = importlib.util.spec_from_file_location("gen_gemm_kloop", os.path.join(os.path.dirname(H.GEMM_SOURCE), "gen_gemm_kloop.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    return {c.name: c for c in gen.SMALL}


def test_launches_of_the_bit_test_end_at_every_place_of_each_ring(loops):
    from tests.test_gpu_ops import TILE_LAUNCHES
    for kind, (loop, launches) in TILE_LAUNCHES.items():
        for glu in {l[0] for l in launches}:
            slices = [k for g, _, _, k in launches if g == glu]
            assert all(H.gemm_plan(M, N, 64 * k, glu) == [(M, kind)] for g, M, N, k in launches if g == glu), kind
            if loop in loops:                                # the big tile's loop is none of the small ones
                c = loops[loop]
                period = sum("v_mfma" in line for line in c.text()) // (2 * c.NS)       # slices of a turn; 2 NS products in each
                assert {(k - 1) % period for k in slices if k > period} == set(range(period)), (kind, glu)


def test_tiles_for_few_rows_keep_their_slices_in_flight(loops):
    """A launch of a few rows streams its weights from memory; the slices requested ahead are what it covers that latency with."""
    for name, in_flight in (("32x32_9", 7), ("64x32_7", 5), ("32x64_4", 3), ("64x64_5", 4)):
        c = loops[name]
        body = c.text()[c.text().index("L_loop_%=:"):]
        wait = next(line for line in body if "vmcnt(" in line)
        left = int(wait.split("vmcnt(")[1].split(")")[0])    # of the loads requested before a barrier, those it does not wait for
        assert left // c.L + 1 == in_flight, name            # and the slice requested behind it
