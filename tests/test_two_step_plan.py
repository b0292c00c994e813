"""How launches are planned (two_step_plan, default_tile), without a GPU: a small
program linked to the library prints the plan of given grids."""
import os
import shutil
import subprocess

import pytest

from paper_1810_09299_amd import abi

HERE = os.path.dirname(os.path.abspath(__file__))
UNIT, MRT, SRT, NMRT = 1, 0, 2, 3              # COLLIDE_*

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None or not os.path.exists(abi.LIB_PATH),
                                reason="needs hipcc and the built library")


@pytest.fixture(scope="module")
def plan_of(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_rules")
    subprocess.run(["hipcc", "-O1", "-std=c++17", "-x", "hip", "--offload-arch=gfx950", "-Xclang", "-target-feature",
                    "-Xclang", "-packed-fp32-ops", os.path.join(HERE, "plan_rules.cpp"), "-x", "none", abi.LIB_PATH,
                    f"-Wl,-rpath,{os.path.dirname(abi.LIB_PATH)}", "-o", exe],
                   check=True, capture_output=True, text=True, timeout=300)

    def plan(precision, grids, alone=False, mode=UNIT):
        line = f"{int(alone)} {abi.PRECISIONS[precision]} {mode} {len(grids)} "
        line += " ".join(f"{nr} {nz} {int(zper)}" for nr, nz, zper in grids)
        r = subprocess.run([exe], input=line, check=True, capture_output=True, text=True, timeout=60)
        march, waves, rows, tile, single_rows = map(int, r.stdout.split())
        return {"march": bool(march), "waves": waves, "rows": rows, "tile": tile, "single_rows": single_rows}

    return plan


@pytest.mark.parametrize("precision,resident", [("fp32", 12), ("fp64", 4)])
@pytest.mark.parametrize("nr,nz", [(9600, 128), (19200, 64), (75000, 16), (300000, 4), (2 ** 23, 4)])
def test_tall_narrow_cases_fill_the_device(plan_of, precision, resident, nr, nz):
    """One strip: the runs of rows are what fills the device's resident wavefronts."""
    p = plan_of(precision, [(nr, nz, True)], alone=True)
    assert p["march"] and p["rows"] >= 4
    assert nz <= 64 * p["waves"]
    slots = 256 * (resident // p["waves"])
    assert -(-nr // p["rows"]) >= slots // 2


def _strips(nz, zper, waves):
    lanes = 64 * waves
    if nz == lanes if zper else nz <= lanes:
        return 1
    return -(-nz // (lanes - 10))


BATCHES = [[(256, 512, True)] * n for n in (7, 9, 10, 11, 16, 20, 33, 64)] + [
    [(512, 2048, True), (32, 64, True)], [(300, 700, False)] * 5 + [(64, 300, True)] * 9,
    [(200, 100, True), (90, 333, True)] * 31, [(128, 512, True)] * 13 + [(255, 509, False)] * 4]


@pytest.mark.parametrize("precision,resident", [("fp32", 12), ("fp64", 4)])
@pytest.mark.parametrize("grids", BATCHES)
def test_march_of_a_batch_goes_by_its_fullest_xcd(plan_of, precision, resident, grids):
    """Runs of rows go to the eight XCDs in turn, all strips of a run to one: no
    other run length would have the fullest XCD done sooner (a run costs ten
    rows beside its own)."""
    p = plan_of(precision, grids)
    if not p["march"]:
        return

    def cost(rows):
        load, nxt = [0] * 8, 0
        for nr, nz, zper in grids:
            for _ in range(-(-nr // rows)):
                load[nxt] += _strips(nz, zper, p["waves"])
                nxt = (nxt + 1) % 8
        return -(-max(load) // (32 * (resident // p["waves"]))) * (rows + 10)

    tallest = max(g[0] for g in grids)
    best = min(cost(-(-tallest // c)) for c in range(1, tallest // 4 + 1))
    assert cost(p["rows"]) == min(best, cost(4))


# us a step as measured on an MI355X: single steps, tiles of 8 x 4, 12 x 8, 16 x 16, 32 x 16 (marching)
MEASURED = [
    ("fp64", NMRT, [(256, 1024, True)], True, (17.3, 46.5, 19.04, 20.67, 17.32)),
    ("fp64", MRT, [(512, 1024, True)], True, (35.86, 91.37, 35.55, 39.18, 33.45)),
    ("fp64", NMRT, [(400, 700, True)], True, (25.76, 49.87, 20.25, 23.96, 22.63)),
    ("fp64", NMRT, [(256, 512, True)] * 4, False, (36.23, 93.63, 37.46, 41.04, 33.96)),
    ("fp64", MRT, [(256, 512, True)] * 6, False, (52.11, 142.39, 56.01, 64.57, 52.88, 48.76)),
    ("fp64", MRT, [(100, 200, True)] * 30, False, (51.42, 117.78, 49.21, 61.1, 57.71, 42.03)),
    ("fp64", SRT, [(256, 512, True)] * 6, False, (51.03, 119.46, 51.8, 42.78, 49.79)),
    ("fp64", UNIT, [(512, 1024, True)], True, (36.14, 76.27, 32.4, 26.29, 31.46)),
    ("fp32", NMRT, [(512, 1024, True)], True, (20.18, 55.78, 23.1, 19.04, 16.61)),
    # the tiles of a batch fill the first XCD before the others
    ("fp32", UNIT, [(42, 896, True)] * 3, False, (9.28, 15.29, 8.6, 7.12, 9.1)),
    ("fp64", UNIT, [(42, 896, True)] * 3, False, (15.02, 22.99, 12.64, 9.98, 15.74)),
    ("fp32", NMRT, [(16, 288, True)] * 20, False, (9.72, 14.74, 8.44, 8.87, 11.4)),
    ("fp64", UNIT, [(16, 288, True)] * 20, False, (15.34, 19.88, 10.5, 10.26, 16.01)),
    # 64 x 8 tiles of single steps fit one to a unit where the smaller ones do not
    ("fp32", UNIT, [(200, 640, True)], True, (6.3, 14.47, 7.51, 7.78, 8.13)),
    ("fp64", UNIT, [(200, 640, True)], True, (9.72, 21.14, 11.14, 11.5, 13.69)),
    ("fp64", SRT, [(69, 1717, True)], True, (11.74, 23.28, 11.82, 12.13, 15.47)),
    ("fp32", NMRT, [(69, 1717, True)], True, (7.83, 16.97, 8.89, 9.48, 9.68)),
    ("fp32", NMRT, [(166, 448, True)], True, (5.78, 11.08, 6.43, 6.68, 6.22)),
    ("fp32", UNIT, [(63, 2047, True)], True, (7.98, 15.92, 8.17, 6.64, 6.26)),
    # the same in a batch of few cases
    ("fp32", UNIT, [(69, 1717, True)], False, (8.04, 15.67, 8.46, 8.84, 8.96)),
    ("fp64", UNIT, [(133, 920, True)], False, (10.54, 22.96, 11.99, 11.82, 14.58)),
    ("fp32", NMRT, [(125, 784, True)], False, (6.36, 14.4, 7.85, 7.31, 6.7)),
    ("fp32", UNIT, [(382, 224, True)], False, (5.81, 11.01, 6.1, 6.05, 6.05)),
    ("fp32", UNIT, [(30, 208, True)] * 14, False, (8.66, 13.48, 7.3, 7.93, 7.37)),
    # small cases, most of their tiles at a rim
    ("fp32", UNIT, [(26, 96, True)] * 161, False, (24.29, 51.93, 26.62, 26.72, 26.89, 21.93)),
    ("fp32", NMRT, [(24, 400, False)] * 59, False, (28.24, 68.96, 28.95, 32.37, 34.19, 26.14)),
    ("fp64", MRT, [(63, 608, True)] * 8, False, (24.92, 63.95, 26.55, 27.74, 27.16, 29.05)),
    ("fp64", MRT, [(46, 176, True)] * 80, False, (59.17, 137.74, 58.65, 68.28, 73.81, 44.19)),
    ("fp64", NMRT, [(278, 128, True)] * 12, False, (33.11, 79.96, 33.32, 35.55, 33.65, 29.22)),
]


@pytest.mark.parametrize("precision,mode,grids,alone,us", MEASURED)
def test_tiles_follow_the_measured_times(plan_of, precision, mode, grids, alone, us):
    """The plan loses no more than the cost model's error (5 %) to single steps,
    and no more than twice that to the best tile shape."""
    p = plan_of(precision, grids, alone=alone, mode=mode)
    got = us[5] if p["march"] else us[p["tile"] + 1]
    assert got <= 1.05 * us[0]
    assert got <= 1.1 * min(us[:5])


# FP16-deviation storage, us a step as measured in 64 x 4 and 64 x 8 tiles
HALF = [(UNIT, 150, 300, True, 5.6, 6.1), (UNIT, 200, 65, True, 8.2, 7.6), (UNIT, 200, 72, False, 8.2, 7.5),
        (SRT, 60, 321, False, 8.4, 7.3), (MRT, 200, 68, True, 9.3, 8.2), (MRT, 160, 328, False, 8.9, 7.8),
        (NMRT, 60, 344, False, 6.5, 6.2), (NMRT, 200, 48, True, 6.3, 6.1), (MRT, 160, 380, True, 6.0, 6.4),
        (UNIT, 256, 512, True, 6.3, 6.0)]


@pytest.mark.parametrize("mode,nr,nz,zper,four,eight", HALF)
def test_fp16_default_tile_follows_the_measured_times(plan_of, mode, nr, nz, zper, four, eight):
    rows = plan_of("fp16", [(nr, nz, zper)], alone=True, mode=mode)["single_rows"]
    assert rows == (4 if four < eight else 8)
