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


@pytest.mark.parametrize("net", [0.0, 3.0])
@pytest.mark.parametrize("levels", [2, 5])
def test_energy_of_charges_between_fp32_numbers(fmm, levels, net):
    # charges s (1 + d), d = 2^-25, are s in FP32; the energy of the exact ones is
    # (1 + d)^2 that of s, where FP32 potentials alone would give 1 + d
    n, box, d = 2000, 20.0, 2.0 ** -25
    pos, _ = workloads.random_charges(n, box, seed=11, net=0.0)
    s = np.where(np.arange(n) % 2 == 0, 1.0, -1.0)
    s[0] += net
    assert np.all((s * (1 + d)).astype(np.float32) == s)
    plan = fmm.fmm_plan(box, levels, 6)
    fmm.fmm_plan_config(plan, fmm.FMM_MIXED)
    e1, _, phi = fmm.fmm_energy_forces(plan, _t(pos), _t(s), phi=True)
    e2, _, _ = fmm.fmm_energy_forces(plan, _t(pos), _t(s * (1 + d)))
    scale = 0.5 * float(np.abs(s) @ np.abs(phi.cpu().numpy()))
    # 2,000 FP64 terms of that total size, rounded once each, and d^2
    assert abs(e2 - e1 * (1 + 2 * d)) < 1e-13 * scale, (e2 / e1 - 1) / d
