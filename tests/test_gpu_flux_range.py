"""The detailed model over the whole range of its fluxes: a state whose pressure, and with it
density, momentum, energy and every flux, is scaled by a power of two, up to flux differences
of about 1e30, where the product of the squared smoothness indicators of both sides of an
interface leaves the range of FP64 unless the fluxes are scaled down. Quarter tiles, whole tiles
with and without components left over, and 1-D tiles; at 2^29 the scaling begins between tiles.

Bar: the repository's 1e-10 per conserved field (and T) against the oracle, which divides for
every candidate; tile widths agree bitwise.
"""

import numpy as np
import pytest

import oracle
from cases import BC_DIRICHLET, BC_SLIPWALL, BC_ZEROGRAD
from gpu_util import rel_err, run_blocks, run_uniform
from test_gpu_stage_tiles import TOL, as_blocks, detailed_state

pytestmark = pytest.mark.gpu


def scaled(ns, nx, ny, power):
    c = detailed_state(ns, nx, ny, [BC_ZEROGRAD, BC_DIRICHLET, BC_SLIPWALL, BC_SLIPWALL], inflow=True)
    s = 2.0 ** power
    c.W[0] *= s
    c.bc_prim[1][0] *= s
    return c


@pytest.mark.parametrize("ns,nx,ny", [(9, 37, 21), (3, 145, 131), (9, 145, 131), (5, 17000, 1)])
@pytest.mark.parametrize("power", [20, 29, 45, 75])
def test_scaled_states(ns, nx, ny, power):
    c = scaled(ns, nx, ny, power)
    Ug, Tg, _, _ = run_uniform(c, 2)
    Uo, To = oracle.case_state(c)
    Uo, To, _, _, _ = oracle.step(c, Uo, To, 2)
    assert np.all(rel_err(Ug, Uo) <= TOL), rel_err(Ug, Uo)
    assert rel_err(Tg[None], To[None])[0] <= TOL


@pytest.mark.parametrize("power", [29, 45])
def test_tile_widths_agree_bitwise(power):
    bc = as_blocks(scaled(5, 145, 131, power))
    ref = run_blocks(bc, 2, tile=16)
    for tile in (32, 64):
        for a, b in zip(run_blocks(bc, 2, tile=tile), ref):
            assert np.array_equal(a, b), tile
