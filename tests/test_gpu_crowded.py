"""Few crowded leaves: the near field with more than 8 wavefronts a leaf, against the
oracle's direct sums in 64 bits.  The chunks that the near field chooses by itself."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _t(a):
    import torch
    return torch.tensor(np.ascontiguousarray(a), device="cuda")


def _rms_rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b)
    return np.sqrt(np.mean((a - b) ** 2) / np.mean(b ** 2))


# 9 to 64 parts a leaf, a leaf of more targets than its parts take at once, and empty ones
@pytest.mark.parametrize("levels,n", [(1, 600), (1, 1601), (1, 4500), (2, 5000), (2, 9000)])
@pytest.mark.parametrize("prec,tol_phi,tol_field", [(0, 1e-14, 1e-14), (1, 1e-6, 2e-6)])
def test_crowded_leaves(fmm, levels, n, prec, tol_phi, tol_field):
    # tolerances of the near field's other tests; FP32 fields grow with the root of the
    # number of sources (7,500 there, up to 70,000 here)
    rng = np.random.default_rng(700 + n)
    box = 20.0
    k = int(np.ceil((2 * n) ** (1 / 3)))
    site = rng.choice(k ** 3, n, replace=False)
    ijk = np.stack([site // (k * k), site // k % k, site % k], 1)
    pos = (ijk + 0.5 + rng.uniform(-0.1, 0.1, (n, 3))) * (box / k)
    if levels == 2:
        pos = pos * [0.74, 1.0, 1.0]  # a quarter of the leaves empty
    q = rng.uniform(-1, 1, n)
    plan = fmm.fmm_plan(box, levels, 2)
    fmm.fmm_plan_config(plan, prec)
    pn, fn, _, _ = fmm.fmm_potential_parts(plan, _t(pos), _t(q))
    phi, field = oracle.nearfield(pos, q, box, levels)
    ep, ef = _rms_rel(pn.cpu().numpy(), phi), _rms_rel(fn.cpu().numpy(), field)
    print(f"levels {levels} n {n} prec {prec}: phi {ep:.2e}, field {ef:.2e}")
    grow = max(1.0, (125 * n / 8 ** levels / 7500) ** 0.5)
    assert ep < tol_phi * grow and ef < tol_field * grow


@pytest.mark.parametrize("levels,n", [(2, 300), (2, 1900), (3, 15000), (4, 60000), (4, 123000)])
def test_default_is_among_the_autotuners_choices(fmm, levels, n):
    # 5 to 30 atoms a leaf, few and many leaves: the order of sums tells the chunk, and
    # that of the default is one of those that the autotuner times
    rng = np.random.default_rng(levels)
    pos, q = rng.uniform(0, 30.0, (n, 3)), rng.uniform(-1, 1, n)
    plan = fmm.fmm_plan(30.0, levels, 2)
    fmm.fmm_plan_config(plan, fmm.FMM_MIXED)
    field = {}
    for g in (0, 2, 4, 8):
        fmm.fmm_plan_tuning(plan, p2p_groups=g)
        field[g] = fmm.fmm_potential_parts(plan, _t(pos), _t(q))[1]
    same = [g for g in (2, 4, 8) if bool((field[0] == field[g]).all())]
    print(f"levels {levels} n {n}: as {same}")
    assert same
