"""Ensembles of many blocks of up to 16 x 8 or 128 x 1 cells (more than 512 tiles), whose stages run
on tiles of 128 cells: bitwise equal to the same domains beside a larger one, which takes the plan
to whole tiles, in other launch forms and at every tile width; and against the oracle at the
repository's 1e-10.
"""

import numpy as np
import pytest

import oracle
import paper_2504_13750_amd as janc
from cases import MODEL_CPG, MODEL_DETAILED, MODEL_ONESTEP
from gpu_util import rel_err, run_blocks
from test_gpu_stage_tiles import TOL
from test_gpu_tiny_blocks import ensemble

pytestmark = pytest.mark.gpu
D1 = [(128, 1), (100, 1), (65, 1), (3, 1), (127, 1)] * 110
D2 = [(16, 8), (10, 6), (9, 3), (3, 8)] * 140
WIDE = [(20, 5), (40, 8), (17, 8), (5, 3)] * 80


@pytest.mark.parametrize("model,ns,sizes", [
    (MODEL_DETAILED, 9, D1), (MODEL_DETAILED, 9, D2), (MODEL_DETAILED, 2, D2), (MODEL_DETAILED, 3, WIDE),
    (MODEL_DETAILED, 4, D1[:300] + D2[:300]), (MODEL_ONESTEP, 0, D2 + [(100, 1)]), (MODEL_ONESTEP, 0, WIDE),
    (MODEL_CPG, 0, D2), (MODEL_CPG, 0, WIDE + [(70, 1)]),
])
def test_blocks_of_half_a_tile(model, ns, sizes):
    n = sum(nx * ny for nx, ny in sizes)
    case = ensemble(model, ns, sizes)
    U, T, t = run_blocks(case, 3)
    whole = run_blocks(ensemble(model, ns, sizes + [(20, 20)]), 3)
    for a, b in zip((U, T, t), (whole[0][:, :n], whole[1][:n], whole[2][:-1])):
        assert np.array_equal(a, b)
    for kw in (dict(flags=janc.PLAN_RESOLVE_HALOS), dict(flags=janc.PLAN_PER_LEVEL), dict(tile=32), dict(tile=64)):
        for a, b in zip(run_blocks(case, 3, **kw), (U, T, t)):
            assert np.array_equal(a, b), kw
    Uo, To = oracle.block_state(case)
    Uo, To, _, _, _ = oracle.step_blocks(case, Uo, To, 3)
    assert np.all(rel_err(U, Uo) <= TOL), rel_err(U, Uo)
    assert rel_err(T[None], To[None])[0] <= TOL


@pytest.mark.parametrize("model", [MODEL_ONESTEP, MODEL_CPG])
def test_one_dimensional_domains_of_half_a_tile(model):
    """Launches per level and stage (in one launch such domains take the kernel of whole runs)."""
    case = ensemble(model, 0, D1)
    ref = run_blocks(case, 3)
    for a, b in zip(run_blocks(case, 3, flags=janc.PLAN_PER_LEVEL), ref):
        assert np.array_equal(a, b)
