"""How launches of two steps are planned (two_step_plan), without a GPU: a small
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
        line = f"{int(alone)} {int(precision == 'fp64')} {mode} {len(grids)} "
        line += " ".join(f"{nr} {nz} {int(zper)}" for nr, nz, zper in grids)
        r = subprocess.run([exe], input=line, check=True, capture_output=True, text=True, timeout=60)
        march, waves, rows, tile = map(int, r.stdout.split())
        return {"march": bool(march), "waves": waves, "rows": rows, "tile": tile}

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
