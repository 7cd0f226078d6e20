"""Ensembles of many tiny blocks (up to 8 x 8 or 64 x 1 cells, more than 64 tiles), whose stages
run on tiles of 64 cells: bitwise equal to the same domains beside a larger one, which takes the
plan to whole tiles, with and without the halo table and with a launch per block; and against
the oracle at the repository's 1e-10.
"""

import numpy as np
import pytest

import oracle
import paper_2504_13750_amd as janc
from cases import (BlockCase, Domain, MODEL_CPG, MODEL_DETAILED, MODEL_ONESTEP, BC_DIRICHLET, BC_PERIODIC,
                   BC_SLIPWALL, BC_ZEROGRAD)
from cases.common import make_blocks
from gpu_util import rel_err, run_blocks
from test_gpu_stage_tiles import TOL, detailed_state

pytestmark = pytest.mark.gpu
BCS = [[BC_ZEROGRAD, BC_DIRICHLET, BC_SLIPWALL, BC_SLIPWALL], [BC_SLIPWALL, BC_ZEROGRAD, BC_PERIODIC, BC_PERIODIC],
       [BC_PERIODIC] * 4]


def ensemble(model, ns, sizes):
    doms, recs, W, mech = [], [], [], None
    rng = np.random.default_rng(5)
    for d, (nx, ny) in enumerate(sizes):
        bc = BCS[d % 3]
        if model == MODEL_DETAILED:
            c = detailed_state(ns, nx, ny, bc, inflow=bc[1] == BC_DIRICHLET)
            w, mech, h, prim = c.W.reshape(ns + 3, -1), c.mech, c.dx, c.bc_prim
            w[0] *= 1.0 + 0.1 * rng.uniform(size=nx * ny)
        else:
            w = np.zeros((5 if model == MODEL_ONESTEP else 4, nx * ny))
            w[0] = 1.0 + 0.3 * rng.uniform(-1, 1, nx * ny)
            w[1], w[2] = 0.2 * rng.uniform(-1, 1, (2, nx * ny))
            w[3] = (8.0 if model == MODEL_ONESTEP else 1.0) * (1.0 + 0.3 * rng.uniform(-1, 1, nx * ny))
            if model == MODEL_ONESTEP:
                w[4] = 0.7
            h, prim = 0.01, [None, w[:, 0].copy() if bc[1] == BC_DIRICHLET else None, None, None]
        recs.append((d, 0, 0, 0, nx, ny))
        doms.append(Domain(nx=nx, ny=ny, dx=h, dy=h, bc=bc, gamma=1.3, Q=20.0, Ea=8.0,
                           k=3.0 if model == MODEL_ONESTEP else 0.0, bc_prim=prim))
        W.append(w)
    return BlockCase(name=f"{len(sizes)} tiny blocks", model=model, domains=doms, blocks=make_blocks(recs),
                     W=np.concatenate(W, axis=1), mech=mech, cfl=0.4)


@pytest.mark.parametrize("model,ns,sizes", [
    (MODEL_DETAILED, 9, [(64, 1), (3, 1), (50, 1), (63, 1), (7, 1)] * 15),
    (MODEL_DETAILED, 3, [(8, 8), (3, 3), (8, 5), (4, 8), (7, 7)] * 15),
    (MODEL_DETAILED, 4, [(8, 8), (64, 1), (3, 8), (20, 1)] * 18),
    (MODEL_ONESTEP, 0, [(8, 8), (3, 4), (5, 8), (8, 3)] * 20),
    (MODEL_CPG, 0, [(8, 8), (30, 1), (6, 7)] * 30),
])
def test_tiny_blocks(model, ns, sizes):
    n = sum(nx * ny for nx, ny in sizes)
    case = ensemble(model, ns, sizes)
    U, T, t = run_blocks(case, 3)
    whole = run_blocks(ensemble(model, ns, sizes + [(20, 20)]), 3)
    for a, b in zip((U, T, t), (whole[0][:, :n], whole[1][:n], whole[2][:-1])):
        assert np.array_equal(a, b)
    for flags in (janc.PLAN_RESOLVE_HALOS, janc.PLAN_PER_BLOCK):
        for a, b in zip(run_blocks(case, 3, flags=flags), (U, T, t)):
            assert np.array_equal(a, b), flags
    Uo, To = oracle.block_state(case)
    Uo, To, _, _, _ = oracle.step_blocks(case, Uo, To, 3)
    assert np.all(rel_err(U, Uo) <= TOL), rel_err(U, Uo)
    assert rel_err(T[None], To[None])[0] <= TOL


@pytest.mark.parametrize("model,ns", [(MODEL_DETAILED, 3), (MODEL_ONESTEP, 0)])
@pytest.mark.parametrize("sizes", [[(8, 8), (5, 7), (8, 5), (3, 4)], [(8, 4), (5, 3)]])
def test_tiny_blocks_at_every_tile_width(model, ns, sizes):
    """64 x 4 tiles: a block of 5 to 8 rows takes two of them, and a tile of 64 cells at the
    first would sweep the rows of both; blocks of up to 4 rows take one."""
    case = ensemble(model, ns, sizes * 20)
    ref = run_blocks(case, 3)
    for tile in (32, 64):
        for a, b in zip(run_blocks(case, 3, tile=tile), ref):
            assert np.array_equal(a, b), tile
