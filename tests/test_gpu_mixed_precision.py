"""What the mixed mode computes in FP64, by its distance from the FP64 mode on one plan."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _t(a):
    import torch
    return torch.tensor(np.ascontiguousarray(a), device="cuda")


@pytest.mark.parametrize("n,box,levels,p", [(4000, 20.0, 5, 4), (20000, 30.0, 5, 6), (20000, 30.0, 5, 3),
                                            (4000, 20.0, 6, 3), (20000, 30.0, 6, 4), (60000, 40.0, 6, 6)])
def test_far_field_of_deep_levels(fmm, n, box, levels, p):
    # levels 1-4 in FP64: what is left is one rounding to FP32 each (2^-24 at most,
    # 3.4e-8 RMS) of the multipoles, the operators, the leaf's locals and the terms of
    # the leaf expansions, independent of each other: 7e-8 if all of the potential came
    # from the finest levels.  Columns or products in FP32 would add as much several times.
    pos, q = workloads.random_charges(n, box, seed=7, net=1.0)
    plan = fmm.fmm_plan(box, levels, p)
    ref = fmm.fmm_potential_parts(plan, _t(pos), _t(q))[2]
    fmm.fmm_plan_config(plan, fmm.FMM_MIXED)
    fmm.fmm_plan_tuning(plan, fp64_levels=4)
    got = fmm.fmm_potential_parts(plan, _t(pos), _t(q))[2]
    err = float((got - ref).norm() / ref.norm())
    print(f"{n} atoms, levels {levels}, p {p}: far-field potential {err:.2e}")
    assert err < 1e-7
