"""GPU parity of the stage kernel on whole tiles (plans of more than 64 tiles; smaller plans run
on quarter tiles): species counts whose component count leaves 0, 1, 2 or 3 over after rounds of
four, of which one or two are swept by all wavefronts together; ragged last tiles; every 2-D tile
width and 1-D tiles.

Bar: the repository's 1e-10 per conserved field (and T) against the oracle; widths agree bitwise.
"""

import numpy as np
import pytest

import oracle
import paper_2504_13750_amd as janc
from cases import BC_DIRICHLET, BC_SLIPWALL, BC_ZEROGRAD, detonation_tube_case
from gpu_util import context_for, rel_err, run_blocks
from test_gpu_stage_tiles import TOL, as_blocks, detailed_state

pytestmark = pytest.mark.gpu
BC = [BC_ZEROGRAD, BC_DIRICHLET, BC_SLIPWALL, BC_SLIPWALL]


def tiles_of(bc, tile):
    ctx = context_for(bc)
    plan = ctx.plan(janc.domains_of(bc), bc.blocks, bc.pool_cells)
    plan.set_tile(tile)
    n = plan.stats()["tiles"]
    plan.close()
    ctx.close()
    return n


def check(case, nsteps, widths):
    bc = as_blocks(case)
    outs = []
    for w in widths:
        assert tiles_of(bc, w) > 64
        outs.append(run_blocks(bc, nsteps, tile=w))
        for a, b in zip(outs[-1], outs[0]):
            assert np.array_equal(a, b), w
    Uo, To = oracle.block_state(bc)
    Uo, To, _, _, _ = oracle.step_blocks(bc, Uo, To, nsteps)
    assert np.all(rel_err(outs[0][0], Uo) <= TOL), rel_err(outs[0][0], Uo)
    assert rel_err(outs[0][1][None], To[None])[0] <= TOL


@pytest.mark.parametrize("ns", [2, 3, 4, 5, 7, 8, 11])
def test_species_counts_of_every_remainder(ns):
    check(detailed_state(ns, 145, 131, BC, inflow=True), 2, [16, 32, 64])


@pytest.mark.parametrize("ns", [2, 3, 4, 5, 7, 9])
def test_one_dimensional_tiles(ns):
    check(detailed_state(ns, 64 * 256 + 37, 1, BC, inflow=True), 2, [16])


def test_one_step_model():
    check(detonation_tube_case(nx=145, ny=131), 3, [16, 32, 64])
    check(detonation_tube_case(nx=64 * 256 + 37, ny=1), 3, [16])
