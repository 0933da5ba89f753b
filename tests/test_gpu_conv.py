"""The convolution M2L against the interaction lists on the GPU.  The symmetric
solute-solvent scheme takes the masked charges' far field through the plan's M2L
(the convolution), the sparse one through the FP64 list operators; both give
sum_u q phi_u and the same e_uv up to the order of FP64 sums, so in FP64 they
agree to rounding at every depth and order: sizes 2 .. 64 of the line transforms,
one to ten row tiles (four and fewer wavefronts), the last one ragged."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _t(a):
    import torch
    return torch.tensor(np.ascontiguousarray(a), device="cuda")


@pytest.mark.parametrize("levels,p", [(1, 0), (1, 9), (2, 3), (2, 12), (3, 4), (3, 8), (4, 1), (4, 7), (4, 11), (5, 2),
                                      (5, 5), (5, 7), (6, 1), (6, 4)])
def test_symmetric_matches_sparse(fmm, levels, p):
    n, box = 900, 20.0
    pos, q = workloads.random_charges(n, box, seed=40 + levels, net=1.0)
    mask = np.zeros(n, np.uint8)
    mask[::7] = 1
    plan = fmm.fmm_plan(box, levels, p)
    assert fmm.fmm_plan_info(plan)["m2l_conv_levels"] == levels
    tp, tq, tm = _t(pos), _t(q), _t(mask)
    got = []
    for scheme in (fmm.FMM_UV_SYMMETRIC, fmm.FMM_UV_SPARSE):
        print(f"levels {levels} p {p} scheme {scheme}", flush=True)
        fmm.fmm_plan_options(plan, fmm.FMM_BOUNDARY_CONDUCTING, scheme)
        _, _, phi = fmm.fmm_energy_forces(plan, tp, tq, forces=False, phi=True)
        got.append(fmm.fmm_solute_solvent_energy(plan, tm))
    unit = float(np.abs(q[mask == 1]).sum()) * float((phi ** 2).mean().sqrt())
    # 900 potentials of about 1e5 FP64 terms each (rounding grows as the root)
    assert abs(got[0] - got[1]) < 1e-12 * unit, (got, unit)


@pytest.mark.parametrize("levels,p", [(3, 6), (4, 10), (5, 4)])
def test_one_crowded_leaf(fmm, levels, p):
    # every atom in one leaf: the transforms spread one cell's expansion over all
    # wave numbers and have to bring zero back elsewhere; FP64 against mixed, and
    # a repeat on the same plan, in place of any other reference
    box = 20.0
    rng = np.random.default_rng(5)
    h = box / 2 ** levels
    pos = np.array([0.25, 0.5, 0.75]) * box + rng.uniform(0.05 * h, 0.95 * h, size=(300, 3))
    q = rng.uniform(-1.0, 1.0, size=300)
    plan = fmm.fmm_plan(box, levels, p)
    e64, f64, _ = fmm.fmm_energy_forces(plan, _t(pos), _t(q))
    again = fmm.fmm_energy_forces(plan, _t(pos), _t(q))
    assert again[0] == e64 and bool((again[1] == f64).all())
    fmm.fmm_plan_config(plan, fmm.FMM_MIXED)
    e32, f32, _ = fmm.fmm_energy_forces(plan, _t(pos), _t(q))
    assert abs(e32 - e64) < 1e-5 * abs(e64)
    assert float((f32 - f64).norm() / f64.norm()) < 1e-5
