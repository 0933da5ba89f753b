"""The near field at the edges of its chunks, and leaves past the sort's in-LDS
capacity, on the GPU against the oracle's direct sums in 64 bits."""
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


def _leaf_atoms(rng, counts, box, levels):
    """counts[c] atoms in cell c (x, y, z order) of the leaf grid, on distinct
    sites of a sub-grid of the cell, jittered by a tenth of its spacing."""
    m = 1 << levels
    h = box / m
    k = int(np.ceil(max(counts) ** (1.0 / 3.0)))
    pos = []
    for c, cnt in enumerate(counts):
        site = rng.permutation(k ** 3)[:cnt]
        ijk = np.stack([site // (k * k), site // k % k, site % k], 1)
        cell = np.array([c // (m * m), c // m % m, c % m])
        pos.append(h * (cell + (ijk + 0.5 + rng.uniform(-0.1, 0.1, (cnt, 3))) / k))
    return np.concatenate(pos)


# target counts around every chunk length (8, 16, 32, 64), around the group counts
# of the sources and around a second chunk of one wavefront, with empty leaves
EDGES = [0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 24, 25, 31, 32, 33, 40, 41, 48, 49, 63, 64, 65, 72, 73, 96, 97, 127,
         128, 129, 0]


@pytest.mark.parametrize("prec,tol_phi,tol_field", [(0, 1e-14, 1e-14), (1, 1e-6, 2e-6)])
@pytest.mark.parametrize("groups", [1, 2, 4, 8, 16])
def test_chunk_edges(fmm, groups, prec, tol_phi, tol_field):
    # the tolerances of the near field's other tests, whose targets have up to 7,500
    # sources each; here they have about 5,800
    rng = np.random.default_rng(600 + groups)
    box, levels = 20.0, 2
    pos = _leaf_atoms(rng, rng.permutation(EDGES * 2), box, levels)
    q = rng.uniform(-1, 1, len(pos))
    plan = fmm.fmm_plan(box, levels, 2)
    fmm.fmm_plan_config(plan, prec)
    fmm.fmm_plan_tuning(plan, p2p_groups=groups)
    pn, fn, _, _ = fmm.fmm_potential_parts(plan, _t(pos), _t(q))
    phi, field = oracle.nearfield(pos, q, box, levels)
    ep, ef = _rms_rel(pn.cpu().numpy(), phi), _rms_rel(fn.cpu().numpy(), field)
    print(f"groups {groups} prec {prec}: phi {ep:.2e}, field {ef:.2e}")
    assert ep < tol_phi and ef < tol_field


@pytest.mark.parametrize("count", [1024, 1025, 1500])
def test_leaf_past_the_sort_capacity(fmm, count):
    # the atoms of the crowded leaf come in a shuffled order; sorted results are put
    # back in the caller's, so a wrong order of any one shows
    rng = np.random.default_rng(count)
    box, levels = 20.0, 2
    counts = np.full(64, 2)
    counts[21] = count
    pos = _leaf_atoms(rng, counts, box, levels)
    pos = pos[rng.permutation(len(pos))]
    q = rng.uniform(-1, 1, len(pos))
    plan = fmm.fmm_plan(box, levels, 2)
    pn, fn, _, _ = fmm.fmm_potential_parts(plan, _t(pos), _t(q))
    phi, field = oracle.nearfield(pos, q, box, levels)
    assert _rms_rel(pn.cpu().numpy(), phi) < 1e-14 and _rms_rel(fn.cpu().numpy(), field) < 1e-14
