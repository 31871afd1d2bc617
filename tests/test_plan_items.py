"""The item split and the tile order of the host planner (hb_plan.cpp, no HIP):
small decode batches are cut finely enough to use the chip, and tiles alone on
the chip are paired longest with shortest."""
import pytest

from test_plan import SHAPES, check, driver, run_plan  # noqa: F401


@pytest.mark.parametrize("name,reqs,units", [
    ("8b", [(1, 1501)], (24, 64)),                           # the smallest range per wave, 64 keys
    ("8b", [(1, 8192)] * 4, (160, 256)),
    ("70b-tp8", [(1, c) for c in (7252, 7089, 598, 647, 5192, 1200, 3000, 4100)], (64, 256)),
    ("g16", [(1, 70), (1, 0), (2, 4000)], (8, 256)),         # hd 64, 16 q heads per kv head
    ("tiny", [(1, 63), (1, 64), (1, 65), (1, 127), (1, 128)], (1, 16)),
    ("8b", [(1, 2300)] * 256, (2048, 2048)),                 # many keys: whole decodes again
])
def test_item_split_fills_the_chip(driver, name, reqs, units):  # noqa: F811
    plan = run_plan(driver, SHAPES[name], 256, reqs)
    check(plan, SHAPES[name], reqs)
    assert units[0] <= len(plan["unit"]) <= units[1], len(plan["unit"])
    assert 64 <= plan["T"][0][2] and plan["T"][0][2] % 64 == 0


@pytest.mark.parametrize("chunk,cu", [(2048, 256), (1100, 256), (1024, 256), (700, 64), (2049, 256)])
def test_tiles_alone_pair_longest_with_shortest(driver, chunk, cu):  # noqa: F811
    reqs = [(chunk, 0)]
    plan = run_plan(driver, SHAPES["8b"], cu, reqs)
    check(plan, SHAPES["8b"], reqs)
    work = [(t[6] - t[5]) * t[4] for t in (plan["tile"][u[0]] for u in plan["unit"])]  # keys x positions
    assert work[:cu] == sorted(work[:cu], reverse=True)
    if cu < len(work) <= 2 * cu:
        assert work[cu:] == sorted(work[cu:]) and min(work[:cu]) >= max(work[cu:])
