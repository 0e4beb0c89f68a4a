"""Every kernel of the ring FFTs is run, whatever the plan's cost model prefers.

Which pass a ring length takes moves with the cost model, so a list of lengths
alone says little: the host test asks the planner (tests/ring_plans) what the
lengths here take, and fails when a pass or tile shape that has a kernel is not
among it, or has no plan at all.  The GPU test runs them against the oracle.
"""
import os
import subprocess

import pytest

from test_gpu_transforms import _check_all, _say, _shtx

EXE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "ring_plans", "_build", "ring_plans")

# (ring length, fields[, latitudes: 4]), chosen from the plans of all even lengths up to 16498 as
# a small set that between them has every pass of every kind and radix and
# every tile shape of the general prime pass
RINGS = {
    "fp64": [(30, 1), (36, 1), (64, 1), (80, 1), (96, 1), (112, 1), (146, 1), (194, 23), (256, 1), (326, 1),
             (370, 13), (446, 1), (482, 1), (548, 1), (562, 1), (612, 1), (734, 1), (780, 1), (872, 1), (1024, 1),
             (1028, 1), (1094, 1), (1372, 1), (1482, 5), (1616, 1), (1796, 1), (1948, 1), (2284, 1), (2310, 1),
             (2754, 1), (3028, 1), (3062, 1), (3156, 3), (3902, 3), (3996, 5), (4034, 3), (4810, 3), (5098, 1),
             (5214, 3), (5296, 1), (5532, 1), (5784, 1), (5854, 3), (6918, 1), (8152, 1), (8672, 1), (8942, 1),
             (478, 1), (514, 2), (518, 23, 400), (566, 1), (614, 1), (1082, 1), (1202, 2), (1542, 3), (2306, 1),
             (2966, 1), (3566, 1), (3980, 1), (6566, 1), (6566, 2, 400), (7252, 1), (7410, 1), (9174, 1)],
    "fp32": [(30, 1), (32, 1), (64, 1), (80, 1), (146, 1), (192, 1), (224, 1), (292, 3), (326, 1), (356, 1),
             (370, 13), (382, 1), (386, 1), (482, 1), (548, 1), (614, 1), (654, 1), (684, 1), (1086, 3), (1088, 1),
             (1300, 1), (1372, 1), (1542, 3), (1616, 1), (1622, 1), (1682, 1), (1746, 1), (1796, 1), (1932, 1),
             (2262, 5), (2284, 1), (2304, 1), (2606, 1), (3080, 1), (3150, 1), (3254, 1), (3396, 3), (3602, 1),
             (3902, 3), (3996, 5), (4162, 1), (4286, 1), (4538, 3), (4810, 3), (4890, 1), (4936, 1), (5214, 3),
             (5532, 1), (6762, 1), (8152, 1), (8834, 1), (8942, 1), (14812, 1), (454, 1), (478, 1), (514, 1),
             (514, 2), (662, 8), (1042, 1), (1154, 3), (1202, 2), (1324, 5), (1538, 2), (1876, 13, 400), (3246, 3),
             (3258, 1), (6566, 1), (6914, 1), (7252, 1), (8762, 1), (9174, 1), (11310, 1)],
}


def _rings(prec):
    return [(*r, 4)[:3] for r in RINGS[prec]]


def _ring_plans(*args, **kw):
    if not os.path.exists(EXE):
        pytest.fail(f"{EXE} is not built (run __graft_entry__.build())")
    return subprocess.run([EXE, *args], capture_output=True, text=True, check=True, timeout=300, **kw).stdout


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_every_kernel_has_a_ring(prec):
    code = ("fp64", "fp32").index(prec)
    kernels = set(_ring_plans("kernels").splitlines()[code].split())
    plans = _ring_plans(input="\n".join(f"{code} {n} {f} 0 {nl}" for n, f, nl in _rings(prec))).splitlines()
    assert len(plans) == len(RINGS[prec]) and "refused" not in plans
    assert len(kernels) > 80
    assert sorted(kernels - {w for p in plans for w in p.split()}) == []


# Roots of unity at quarter turns are exact zeros and ones: cosl(pi / 2) is 1e-20,
# and what should cancel would leave that much of the other values.
def test_quarter_turns_are_exact():
    lengths = [24, 64, 244, 488, 1604, 2416, 4996, 5120]
    plans = _ring_plans(input="\n".join(f"{c} {n} 3 0 4" for n in lengths for c in (0, 1))).splitlines()
    assert len(plans) == 2 * len(lengths) and not any("residue" in p for p in plans)


# Few values a block take the kind with the fewest passes, many the one with the
# least work (the faster of the two by 15 to 50 % in each case).
@pytest.mark.parametrize("prec,nlon,nf,want", [
    ("fp64", 244, 2, "gp:61"), ("fp64", 404, 1, "gp:101"), ("fp64", 146, 8, "gp:73"), ("fp32", 122, 3, "gp:61"),
    ("fp32", 610, 1, "gp:61"), ("fp32", 452, 3, "gp:113"), ("fp32", 2416, 200, "conv"), ("fp32", 4036, 100, "conv"),
    ("fp64", 2416, 200, "conv"), ("fp32", 1556, 411, "blue")])
def test_choice_follows_the_size(prec, nlon, nf, want):
    words = _ring_plans(input=f"{('fp64', 'fp32').index(prec)} {nlon} {nf} 0 512").split()
    kinds = {w.split(":")[0] for w in words}
    if want == "conv":
        assert "9" in kinds and "gp" not in kinds
    elif want == "blue":
        assert "5" in kinds
    else:
        assert want in words


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_every_ring_kernel_parity(prec):
    shtx = _shtx()
    for nlon, nf, nlat in _rings(prec):
        n = min(20, (nlon - 1) // 2)
        _say(f"ring kernels nlon={nlon} F={nf} nlat={nlat} {prec}")
        plan = shtx.Plan(n, "full", nlat, nf, prec, nlon_full=nlon)
        _check_all(plan, n, plan.ring_lengths(), 47, range(nf), prec)
        plan.close()
