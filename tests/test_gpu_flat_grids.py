"""Uniform grids of few rows and many columns, whose tile width follows from the padding and the
cost of each width: janc_step and janc_step_noalloc bitwise equal to a block table of the same
grid at every width, at row counts on both sides of the tile heights."""

import numpy as np
import pytest

import paper_2504_13750_amd as janc
from cases import MODEL_DETAILED, MODEL_ONESTEP, BC_DIRICHLET, BC_SLIPWALL, BC_ZEROGRAD, detonation_tube_case
from gpu_util import run_blocks, run_uniform, torch_dev
from test_gpu_stage_tiles import as_blocks, detailed_state

pytestmark = pytest.mark.gpu


def noalloc(c, nsteps):
    torch, dev = torch_dev()
    ctx = janc.Context(c.model, c.mech)
    U, T = ctx.init_state(janc.physics_of(c), torch.tensor(c.W, dtype=torch.float64, device=dev))
    t = torch.zeros(1, dtype=torch.float64, device=dev)
    print(f"[gpu] janc_step_noalloc {c.name} nsteps={nsteps}", flush=True)
    ctx.step_noalloc(janc.grid_of(c), janc.physics_of(c), janc.time_of(c), U, T, nsteps, t)
    ctx.sync_status()
    out = U.cpu().numpy(), T.cpu().numpy()
    ctx.close()
    return out


@pytest.mark.parametrize("ny", [3, 4, 5, 8, 9, 15, 16, 17, 24, 31])
@pytest.mark.parametrize("model,ns", [(MODEL_ONESTEP, 0), (MODEL_DETAILED, 3), (MODEL_DETAILED, 5)])
def test_flat_grids(model, ns, ny):
    nx = 2500
    c = (detonation_tube_case(nx=nx, ny=ny) if model == MODEL_ONESTEP else
         detailed_state(ns, nx, ny, [BC_ZEROGRAD, BC_DIRICHLET, BC_SLIPWALL, BC_SLIPWALL], inflow=True))
    U, T, _, _ = run_uniform(c, 2)
    outs = [noalloc(c, 2)] + [run_blocks(as_blocks(c), 2, tile=w)[:2] for w in (16, 32, 64)]
    for u, t in outs:
        assert np.array_equal(U.ravel(), u.ravel()) and np.array_equal(T.ravel(), t.ravel())
