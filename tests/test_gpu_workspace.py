"""Plans whose workspace or operators are not where the last call left them.  Batches
whose boxes change size between calls: a box's workspace grows and moves,
and every pass has to work on the new one.  The first call of a plan."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _t(a):
    import torch
    return torch.tensor(np.ascontiguousarray(a), device="cuda")


BOXES, LEVELS = [20.0, 21.0, 22.0], [2, 3, 1]


def _inputs(counts, seed):
    parts = [workloads.random_charges(n, b, seed=seed + k, net=1.0) for k, (n, b) in enumerate(zip(counts, BOXES))]
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    mask = np.zeros(off[-1], np.uint8)
    mask[::5] = 1
    return off, _t(np.concatenate([p for p, _ in parts])), _t(np.concatenate([q for _, q in parts])), _t(mask)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("scheme", [0, 1, 2])  # symmetric, sparse, swapped symmetric
def test_batch_uv_after_a_larger_batch(fmm, prec, scheme):
    # small batch, larger batch, the small sizes again with other atoms: bit for
    # bit what a plan that has seen nothing else gives
    a, b, c = _inputs([300, 400, 200], 900), _inputs([6000, 8000, 4000], 910), _inputs([300, 400, 200], 920)

    def plan():
        p = fmm.fmm_plan_batch(BOXES, 4, levels=LEVELS)
        fmm.fmm_plan_config(p, prec)
        fmm.fmm_plan_options(p, fmm.FMM_BOUNDARY_CONDUCTING, scheme)
        return p

    def both(p, x):
        off, pos, q, mask = x
        e, _ = fmm.fmm_energy_forces_batch(p, off, pos, q)
        return e, fmm.fmm_solute_solvent_energy_batch(p, mask)

    used = plan()
    both(used, a)
    fmm.fmm_energy_forces_batch(used, *b[:3])
    got = both(used, c)
    want = both(plan(), c)
    np.testing.assert_array_equal(got[0], want[0])
    np.testing.assert_array_equal(got[1], want[1])


@pytest.mark.parametrize("levels,p", [(4, 14), (3, 20)])
def test_new_plan_without_allocation(fmm, levels, p):
    # operators of more than 1 GiB in FP64: there without another call before
    import torch
    pos, q = workloads.random_charges(500, 20.0, seed=930, net=1.0)
    plan = fmm.fmm_plan(20.0, levels, p)
    f = torch.empty((500, 3), dtype=torch.float64, device="cuda")
    e = fmm.fmm_energy_forces_noalloc(plan, _t(pos), _t(q), forces=f)
    want = fmm.fmm_energy_forces(plan, _t(pos), _t(q))
    assert e == want[0] and bool((f == want[1]).all())
