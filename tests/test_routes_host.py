"""The shapes that the GPU tests name for a kernel are the ones that the dispatch sends there (on 256 compute units): the rule of
mma_types.h, compiled for the host."""
import os
import shutil
import subprocess

import pytest

import test_gpu_fused
import test_gpu_large_tiles
import test_gpu_lifted_tiles
import test_gpu_mid_tiles
import test_gpu_narrow_tiles
import test_gpu_parity
import test_gpu_replay
import test_gpu_slim
import test_gpu_small_tiles
import test_gpu_wide_layers
import test_gpu_y_rows
import test_zz_no_alloc
from paper_2603_05232_amd import binding, build, synth

SOURCE = """
#include "mma_types.h"
#include <stdio.h>
using namespace ss;
int main()
{
    int kind; long long M, O, units; unsigned long long ws;
    while (scanf("%d %lld %lld %lld %llu", &kind, &M, &O, &units, &ws) == 5) {
        const ss_plan p = plan_gemm((ss_kind)kind, M, O, units, (size_t)ws);
        const long long cut = p.path == SS_PATH_TILE ? (long long)p.tile_o : 0;
        const int rest = cut == 0 || cut == O ? -1 : kind == SS_KIND_FUSED && narrow_pays(M, O - cut, cu_count()) ? SS_PATH_NARROW : SS_PATH_MID;
        const bool groups = kind == SS_KIND_LIFTED && p.path == SS_PATH_MID && two_groups(M, O, units, cu_count());
        const bool stream = p.path == SS_PATH_WIDE || (kind != SS_KIND_DENSE && p.path == SS_PATH_MID && M <= 32 && !groups && (O + 127) / 128 * p.S <= cu_count());
        printf("%d %d %lld %d %d %d %d %d %d\\n", (int)p.path, p.S, cut, rest, cu_count(), groups, stream, p.small.fw, p.small.tb);
    }
}
"""
SKINNY, MID, NARROW, TILE, WIDE, SLIM, SMALL = range(7)
LIFTED, FUSED, DENSE = 0, 1, 2


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if shutil.which(hipcc) is None:
        pytest.skip("no hipcc")
    binding.load()
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SOURCE)
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-std=c++17", "-I" + os.path.join(build.ROOT, "include"), "-I" + build.CSRC,
                    "-c", str(d / "plan.cpp"), "-o", str(d / "plan.o")], check=True)
    subprocess.run([hipcc, str(d / "plan.o"), "-L" + build.PKG, "-lslidesparse", "-Wl,-rpath," + build.PKG, "-o", str(d / "plan")], check=True)

    def ask(kind, M, O, units, ws=0):
        out = subprocess.run([str(d / "plan")], input=f"{kind} {M} {O} {units} {ws}\n", stdout=subprocess.PIPE, text=True, check=True).stdout
        path, S, cut, rest, cus, groups, stream, fw, tb = map(int, out.split())
        if cus != 256:
            pytest.skip("the shapes are chosen for 256 compute units")
        return {"path": path, "S": S, "cut": cut, "rest": rest, "groups": bool(groups), "stream": bool(stream), "large_tiles": -(-cut // 256) * -(-M // 256), "small": (fw, tb)}
    return ask


@pytest.mark.parametrize("kind,module", [(FUSED, test_gpu_large_tiles), (LIFTED, test_gpu_lifted_tiles)])
def test_rounds_of_large_tiles(plan, kind, module):
    for M, O, units in module.ROUNDS:
        p = plan(kind, M, O, units)
        assert p["path"] == TILE and p["large_tiles"] > 256, (M, O, units, p)
    assert {u for M, O, u in module.ROUNDS if M == 8100} >= {1, 2, 3, 4, 5}
    for M, O, units in module.ONE_ROUND_AND_REST:
        p = plan(kind, M, O, units)
        assert p["path"] == TILE and p["large_tiles"] <= 256 and p["rest"] == MID, (M, O, units, p)


def test_narrow_tiles(plan):
    for M, O in test_gpu_narrow_tiles.EDGES + [(1100, 4224), (1100, 4221), (700, 50 * 128 - 5)]:
        assert plan(FUSED, M, O, 5)["path"] == NARROW, (M, O)
    M, O = test_gpu_narrow_tiles.REST
    assert plan(FUSED, M, O, 16)["rest"] == NARROW and plan(FUSED, M, O, 15)["cut"] == O


def test_shared_compute_units(plan):
    for dtype, M, O, units, N, fused in test_gpu_mid_tiles.SHARED:
        p = plan(FUSED if fused else LIFTED, M, O, units)
        assert p["path"] == MID and -(-M // 128) * -(-O // 128) > 256, (dtype, M, O, units, N, fused, p)
    for dtype, M, O, units, N, fused in test_gpu_mid_tiles.SHARED_NARROW:
        assert plan(FUSED, M, O, units)["path"] == NARROW


def test_lines_of_the_kernel_choice(plan):
    """Each line of test_gpu_mid_tiles.test_lines_of_the_kernel_choice has a row on either side."""
    for kind, line, many in ((FUSED, 12, 24), (LIFTED, 24, 48)):
        for panels, units in ((321, line), (449, many)):
            assert plan(kind, 65, 128 * panels, units - 1)["path"] == TILE and plan(kind, 65, 128 * panels, units)["path"] == MID
        assert plan(kind, 65, 128 * 320, 3)["path"] == MID and plan(kind, 65, 128 * 513, 48)["path"] == TILE
        for M, panels, path in ((15, 191, SKINNY), (15, 192, MID), (16, 127, SKINNY), (16, 128, MID), (64, 127, SMALL), (64, 128, SMALL)):
            assert plan(kind, M, 128 * panels, 3)["path"] == path, (M, panels)
        for M, line, path in ((1, 64, SLIM), (32, 48, SMALL), (33, 48, SMALL), (64, 48, SMALL)):
            assert plan(kind, M, 500, line - 1, 1 << 30)["path"] == path and plan(kind, M, 500, line, 1 << 30)["S"] > 1, (M, line)


def test_up_to_32_tokens(plan):
    for M, O, units in test_gpu_mid_tiles.TWO_GROUPS:
        assert plan(LIFTED, M, O, units)["groups"], (M, O, units)
        assert not plan(FUSED, M, O, units)["groups"] and not plan(LIFTED, M, O, 11)["groups"]
    assert not plan(LIFTED, 32, 170 * 128 + 1, 40)["groups"] and not plan(LIFTED, 32, 127 * 128, 40)["groups"] and not plan(LIFTED, 15, 129 * 128, 15)["groups"]
    for M, O, units, with_ws in test_gpu_mid_tiles.STREAM:
        for kind in (FUSED, LIFTED):
            p = plan(kind, M, O, units, 1 << 30 if with_ws else 0)
            assert p["stream"] and (p["S"] > 1) == with_ws, (kind, M, O, units)
    for M, O, units in test_gpu_mid_tiles.FEW_TOKENS:
        for kind in (FUSED, LIFTED):
            assert plan(kind, M, O, units)["path"] == SKINNY, (kind, M, O, units)
    for M, O, units in test_gpu_mid_tiles.LONG_ROWS:
        for ws in (0, 1 << 30):
            p = plan(FUSED, M, O, units, ws)
            assert p["path"] == MID and p["stream"] and p["S"] == 1, (M, O, units, p)
            assert plan(FUSED, M, O, 42, ws)["path"] == plan(FUSED, M, 127 * 128, units, ws)["path"] == SMALL


def test_large_weights(plan):
    for M, O, units, fused, limit in test_gpu_mid_tiles.LARGE:
        p = plan(FUSED if fused else LIFTED, M, O, units)
        assert (p["path"], p["S"]) == (MID, 1) and not p["stream"] and not p["groups"], (M, O, units, fused)
        assert limit << 20 <= O * units * (120 if fused else 80) < 2 * limit << 20
        assert (-(-O // 128) > 256) == (O > 512 * 128)                   # shared compute units
    M, O, units = test_gpu_mid_tiles.TWO_GROUPS[-1]
    assert O * units * 80 >= 80 << 20


def test_numbers_of_ranges(plan):
    for M, O, units, S in test_gpu_mid_tiles.RANGES:
        for kind in (FUSED, LIFTED):
            p = plan(kind, M, O, units, 1 << 30)
            assert (p["path"], p["S"]) == (MID, S), (M, O, units, p)


def test_blocks_of_the_reduce_kernel(plan):
    for i, (M, O, units) in enumerate(test_gpu_mid_tiles.BLOCKS):
        for kind in (FUSED, LIFTED):
            p = plan(kind, M, O, units, 1 << 30)
            assert p["path"] == MID and p["S"] > 1 and (-(-M // 128) * -(-O // 128) > 32) == i % 2, (M, O, units, p)


def test_wide_layers(plan):
    for M, O, units, fused in test_gpu_wide_layers.SHAPES:
        assert plan(FUSED if fused else LIFTED, M, O, units)["path"] == WIDE, (M, O, units, fused)
        assert plan(FUSED if fused else LIFTED, M, O, 15)["path"] != WIDE
    for M, O, units, fused in test_gpu_wide_layers.BESIDE:
        assert plan(FUSED if fused else LIFTED, M, O, units)["path"] in (MID, TILE), (M, O, units, fused)
    for kind in (FUSED, LIFTED):
        assert plan(kind, 32, 171 * 128, 16)["path"] == plan(kind, 1, 256 * 128, 16)["path"] == plan(FUSED, 32, 129 * 128, 16)["path"] == WIDE
        assert plan(kind, 33, 256 * 128, 16)["path"] == plan(kind, 5, 513 * 128, 16)["path"] == MID


def test_replayed_routes(plan):
    for name, (fused, M, O, K, with_ws) in test_gpu_replay.ROUTES.items():
        units = (K if fused else binding.slide_lifted_ld(K, 4, "i8")) // 128
        p = plan(FUSED if fused else LIFTED, M, O, units, 1 << 30 if with_ws else 0)
        if "groups" in name:
            assert p["groups"] and not with_ws, name
        elif "panel" in name:
            assert p["path"] == MID and p["stream"] and (p["S"] > 1) == with_ws, name
        elif "sixteen" in name:
            assert p["path"] == SLIM, name
        elif "small tiles" in name:
            assert p["path"] == SMALL and f"{p['small'][0]} x {p['small'][1]}" in name, name
        elif "few-token" in name:
            assert p["path"] == SKINNY, name
        elif "split tiles" in name:
            assert p["path"] == MID and p["S"] > 1 and ("64" in name) == (M <= 64), name
        elif name == "five fragments a workgroup":
            assert p["path"] == WIDE, name
        elif name == "narrow tiles":
            assert p["path"] == NARROW, name
        else:
            assert p["path"] == TILE and (p["rest"] == NARROW) == ("rest" in name) and (p["large_tiles"] > 256) == ("rounds" in name), name
        if "odd" in name or "even" in name:
            assert units % 2 == ("odd" in name), name
        if "short" in name:
            assert units < 4, name


def test_sixteen_channels(plan):
    for kind in (FUSED, LIFTED):
        for M, O, units, with_ws in test_gpu_slim.SHAPES:
            assert plan(kind, M, O, units, 1 << 30 if with_ws else 0)["path"] == SLIM, (kind, M, O, units)
        for M, O, units, with_ws in test_gpu_slim.BESIDE:
            assert plan(kind, M, O, units, 1 << 30 if with_ws else 0)["path"] != SLIM, (kind, M, O, units)


def test_small_tiles(plan):
    for M, O, units, with_ws, fw, tb in test_gpu_small_tiles.SHAPES:
        for kind in (FUSED, LIFTED):
            p = plan(kind, M, O, units, 1 << 30 if with_ws else 0)
            assert p["path"] == SMALL and p["small"] == (fw, tb) and p["S"] == 1, (kind, M, O, units, p)
    for M, O, units, with_ws in test_gpu_small_tiles.BESIDE:
        for kind in (FUSED, LIFTED):
            assert plan(kind, M, O, units, 1 << 30 if with_ws else 0)["path"] != SMALL, (kind, M, O, units)


def test_rows_of_results(plan):
    for shapes, path in ((test_gpu_y_rows.MID, MID), (test_gpu_y_rows.WIDE, WIDE), (test_gpu_y_rows.SMALL, SMALL)):
        for M, O, units in shapes:
            p = plan(FUSED, M, O, units)
            assert p["path"] == path and p["S"] == 1, (M, O, units, p)


def _lifted_units(K, N):
    return binding.slide_lifted_ld(K, N, "i8") // 128


def test_split_rows(plan):
    """The INT8 calls that a test names for split rows are split, those for small tiles are not."""
    many = 1 << 30
    for split, cases in ((True, test_gpu_parity.SPLIT), (False, test_gpu_parity.SPLIT_DENSE)):
        for N, M, O, K in cases:
            p = plan(LIFTED, M, O, _lifted_units(K, N), many)
            assert (p["path"] == MID and p["S"] > 1) if split else p["path"] == SMALL, (N, M, O, K, p)
            if not split:
                assert plan(DENSE, M, O, K // 128, many)["S"] > 1, (M, O, K)
    for cases, split in ((test_zz_no_alloc.CASES, True), (test_zz_no_alloc.UNSPLIT, False)):
        for M, O, K in cases:
            p = plan(LIFTED, M, O, _lifted_units(K, 4), binding.slide_static_scratch_bytes())
            assert (p["path"] == MID and p["S"] > 1) if split else p["path"] == SMALL, (M, O, K, p)
    for kind, cases in ((LIFTED, test_gpu_parity.REPLAYED), (FUSED, test_gpu_fused.REPLAYED)):
        for M, K, split in cases:
            p = plan(kind, M, 640, K // 128 if kind == FUSED else _lifted_units(K, 4), many)
            assert (p["path"] == MID and p["S"] > 1) if split else p["path"] == (SLIM if M == 16 else SMALL), (kind, M, K, p)
    for M in (128, 256):
        for i, expected in ((0, SMALL), (3, MID)):
            name, K, O = synth.QWEN25_7B[i]
            p = plan(LIFTED, M, O, _lifted_units(K, 4), many)
            assert p["path"] == expected and (p["S"] > 1) == (i == 3), (name, M, p)
    for M, O, alone in ((3, 40, SLIM), (65, 16, SMALL)):                    # the longest rows
        assert plan(LIFTED, M, O, 65535)["path"] == alone and plan(LIFTED, M, O, 65535, many)["S"] > 1
