"""The M2L over the interaction lists, where the convolution is held back
(fmm_plan_conv_levels): all levels on the lists, and trees whose upper levels are a
convolution and whose finer ones are lists, as where its operators find no memory.
The reference is the FP64 mode with the convolution on the same tree: the same
truncation, so that what differs is the rounding of the mode.  The convolution itself
at the orders past 12."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

FP64, MIXED, SPLIT16 = 0, 1, 3
# difference from FP64 (energy, forces, potential): rounding of 64-bit sums of up to
# 1e5 terms; the tolerances of the mixed and split modes' other tests
TOL = {FP64: (1e-12, 1e-11, 1e-11), MIXED: (1e-6, 1e-5, 1e-5), SPLIT16: (1e-6, 1e-5, 1e-5)}


def _t(a):
    import torch
    return torch.tensor(np.ascontiguousarray(a), device="cuda")


_box = {}


def _inputs(name):
    if name not in _box:
        if name in ("C1", "C2"):
            w = workloads.config(name)
            _box[name] = (_t(w.pos), _t(w.q), w.box)
        else:
            n, box = {"sparse": (20000, 40.0)}[name]
            pos, q = workloads.random_charges(n, box, seed=77, net=1.0)
            _box[name] = (_t(pos), _t(q), box)
    return _box[name]


def _check(fmm, name, levels, p, prec, cap, fp64_levels=3):
    pos, q, box = _inputs(name)
    plan = fmm.fmm_plan(box, levels, p)
    assert fmm.fmm_plan_info(plan)["m2l_conv_levels"] == levels
    e0, f0, phi0 = fmm.fmm_energy_forces(plan, pos, q, phi=True)
    fmm.fmm_plan_conv_levels(plan, cap)
    fmm.fmm_plan_config(plan, prec)
    fmm.fmm_plan_tuning(plan, fp64_levels=fp64_levels)
    assert fmm.fmm_plan_info(plan)["m2l_conv_levels"] == (cap if cap >= min(4, levels) else 0)
    e, f, phi = fmm.fmm_energy_forces(plan, pos, q, phi=True)
    err = (abs(e - e0) / abs(e0), float((f - f0).norm() / f0.norm()), float((phi - phi0).norm() / phi0.norm()))
    print(f"{name} levels {levels} p {p} prec {prec} lists past {cap}: energy {err[0]:.1e} force {err[1]:.1e} "
          f"potential {err[2]:.1e}")
    assert all(a < b for a, b in zip(err, TOL[prec])), err
    again = fmm.fmm_energy_forces(plan, pos, q)
    assert again[0] == e and bool((again[1] == f).all())
    fmm.fmm_destroy(plan)


# one and two levels, partly filled tiles, every level in the mode's operands
@pytest.mark.parametrize("levels,p", [(1, 8), (2, 8), (1, 12), (2, 12)])
@pytest.mark.parametrize("prec", [FP64, MIXED, SPLIT16])
def test_shallow(fmm, levels, p, prec):
    _check(fmm, "C1", levels, p, prec, 0, fp64_levels=0)


# the layouts of the lists: (t, -t) pairs and orbits, one to seven row blocks a class,
# the plain and the folded split-FP16 kernel in one and two row groups
@pytest.mark.parametrize("p,prec", [(p, MIXED) for p in (2, 4, 7, 9, 10, 12, 14, 16, 20)] +
                         [(p, SPLIT16) for p in (4, 8, 11, 12, 16, 20)] + [(p, FP64) for p in (4, 7, 10, 13, 20)])
def test_layouts(fmm, p, prec):
    _check(fmm, "C2", 4, p, prec, 0, fp64_levels=0)


# lists below a convolution: FP64 locals handed down to FP32 ones, list levels in FP64
# below it, and the whole of a deep tree on the lists
@pytest.mark.parametrize("levels,cap", [(5, 4), (6, 4), (6, 5), (5, 0), (6, 3)])
@pytest.mark.parametrize("p,prec", [(3, FP64), (4, MIXED), (4, SPLIT16), (8, FP64), (8, MIXED), (8, SPLIT16),
                                    (12, MIXED), (12, SPLIT16)])
def test_below_the_convolution(fmm, levels, cap, p, prec):
    _check(fmm, "sparse", levels, p, prec, cap)


def test_fp64_levels_past_the_convolution(fmm):
    _check(fmm, "sparse", 6, 6, MIXED, 4, fp64_levels=5)


def test_levels_seven(fmm):
    # the depth that no convolution reaches
    pos, q, box = _inputs("sparse")
    plan = fmm.fmm_plan(box, 6, 4)
    e0, f0, _ = fmm.fmm_energy_forces(plan, pos, q)
    fmm.fmm_destroy(plan)
    plan = fmm.fmm_plan(box, 7, 4)
    assert fmm.fmm_plan_info(plan)["m2l_conv_levels"] == 6
    got = {}
    for prec in (FP64, MIXED, SPLIT16):
        fmm.fmm_plan_config(plan, prec)
        got[prec] = fmm.fmm_energy_forces(plan, pos, q)
    # another tree: the truncation of the order between the two (1e-4 of the forces)
    assert abs(got[FP64][0] - e0) < 1e-4 * abs(e0) and float((got[FP64][1] - f0).norm() / f0.norm()) < 1e-2
    for prec in (MIXED, SPLIT16):
        assert abs(got[prec][0] - got[FP64][0]) < 1e-6 * abs(e0)
        assert float((got[prec][1] - got[FP64][1]).norm() / f0.norm()) < 1e-5


def test_held_back_batch(fmm):
    # a batch takes it as its boxes would alone, and so does the call that may not allocate
    pos, q, box = _inputs("C1")
    n = q.shape[0]
    single = fmm.fmm_plan(box, 2, 6)
    fmm.fmm_plan_conv_levels(single, 0)
    e, f, _ = fmm.fmm_energy_forces(single, pos, q)
    assert fmm.fmm_energy_forces_noalloc(single, pos, q) == e
    batch = fmm.fmm_plan_batch([box], 6, levels=[2])
    fmm.fmm_plan_conv_levels(batch, 0)
    eb, fb = fmm.fmm_energy_forces_batch(batch, np.array([0, n]), pos, q)
    assert eb[0] == e and bool((fb == f).all())
    for bad in (-1, 7):
        with pytest.raises(fmm.FmmError):
            fmm.fmm_plan_conv_levels(single, bad)


@pytest.mark.parametrize("levels,p", [(2, 20), (3, 16), (3, 20), (4, 13), (5, 14)])
def test_convolution_of_high_orders(fmm, levels, p):
    # 13 to 28 row tiles; FP64 against the lists on the same plan
    _check(fmm, "C1" if levels < 4 else "C2", levels, p, FP64, 0)
