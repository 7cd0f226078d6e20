"""janc_step_noalloc builds the halo source table in its scratch array when a call has several
steps and the table fits beside the state; else its stages look every halo source up. All
forms do the same arithmetic, so they are held to equality with janc_step: one step (no
table), two and more (table), a grid that leaves no room for it (832 x 832 one-step cells take
66.5 of the 67.1 MB), a larger call after a smaller one, and rows that are one tile wide."""

import numpy as np
import pytest

import paper_2504_13750_amd as janc
from cases import detonation_tube_case
from cases.amr import detailed_front_case
from gpu_util import context_for, torch_dev

pytestmark = pytest.mark.gpu


def _run(case, nsteps, noalloc, ctx):
    torch, dev = torch_dev()
    phys = janc.physics_of(case)
    U, T = ctx.init_state(phys, torch.tensor(case.W, dtype=torch.float64, device=dev))
    t = torch.zeros(1, dtype=torch.float64, device=dev)
    step = ctx.step_noalloc if noalloc else ctx.step
    print(f"[gpu] {case.nx}x{case.ny} nsteps={nsteps} noalloc={noalloc}", flush=True)
    step(janc.grid_of(case), phys, janc.time_of(case), U, T, nsteps, t)
    ctx.sync_status()
    return U.cpu().numpy(), T.cpu().numpy(), t.item()


@pytest.mark.parametrize("model,nx,ny,steps", [
    ("onestep", 64, 16, (1, 2, 5)),
    ("onestep", 131, 13, (3, 1, 2)),
    ("onestep", 1500, 3, (2,)),
    ("onestep", 832, 832, (2, 1)),
    ("detailed", 37, 21, (1, 3)),
])
def test_noalloc_with_and_without_the_halo_table(model, nx, ny, steps):
    if model == "onestep":
        c = detonation_tube_case(nx=nx, ny=ny, seed=33)
    else:
        c = detailed_front_case(nx=nx, ny=ny)
    ctx = context_for(c)
    for n in steps:
        (Ur, Tr, tr), (Ug, Tg, tg) = _run(c, n, False, ctx), _run(c, n, True, ctx)
        assert np.array_equal(Ug, Ur) and np.array_equal(Tg, Tr) and tg == tr
    ctx.close()
