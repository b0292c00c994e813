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

    def plan(precision, grids, singly=False, mode=UNIT):
        line = f"{int(singly)} {int(precision == 'fp64')} {mode} {len(grids)} "
        line += " ".join(f"{nr} {nz} {int(zper)}" for nr, nz, zper in grids)
        r = subprocess.run([exe], input=line, check=True, capture_output=True, text=True, timeout=60)
        march, waves, rows, tile = map(int, r.stdout.split())
        return {"march": bool(march), "waves": waves, "rows": rows, "tile": tile}

    return plan


@pytest.mark.parametrize("precision,resident", [("fp32", 12), ("fp64", 4)])
@pytest.mark.parametrize("nr,nz", [(9600, 128), (19200, 64), (75000, 16), (300000, 4), (2 ** 23, 4)])
def test_tall_narrow_cases_fill_the_device(plan_of, precision, resident, nr, nz):
    """One strip: the runs of rows are what fills the device's resident wavefronts."""
    p = plan_of(precision, [(nr, nz, True)], singly=True)
    assert p["march"] and p["rows"] >= 4
    assert nz <= 64 * p["waves"]
    slots = 256 * (resident // p["waves"])
    assert -(-nr // p["rows"]) >= slots // 2
