"""Whole runs of many tiny one-dimensional domains in one launch: sizes on both sides of every
LDS capacity, more domains than the chip holds at once (fewer wave groups per domain, several
turns, fewer steps per launch), and domains of unlike sizes (a launch for each LDS capacity),
bitwise equal to the launches per stage. The dt log of a call of several launches equals that of calls of one launch each.
"""

import numpy as np
import pytest

import paper_2504_13750_amd as janc
from cases import MODEL_CPG, MODEL_ONESTEP, BC_DIRICHLET, BC_PERIODIC, BC_SLIPWALL, BC_ZEROGRAD
from gpu_util import torch_dev
from test_gpu_tiny_runs import domains, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,sizes,bc,nsteps", [
    (MODEL_CPG, [127], (BC_PERIODIC, BC_PERIODIC), 10),
    (MODEL_ONESTEP, [128], (BC_ZEROGRAD, BC_DIRICHLET), 10),
    (MODEL_CPG, [255, 30], (BC_SLIPWALL, BC_DIRICHLET), 10),
    (MODEL_ONESTEP, [256], (BC_PERIODIC, BC_PERIODIC), 10),
    (MODEL_ONESTEP, [511, 64], (BC_SLIPWALL, BC_ZEROGRAD), 10),
    (MODEL_CPG, [512], (BC_ZEROGRAD, BC_DIRICHLET), 10),
    (MODEL_ONESTEP, [512], (BC_ZEROGRAD, BC_DIRICHLET), 10),      # the largest alone and one more
    (MODEL_CPG, [767], (BC_SLIPWALL, BC_DIRICHLET), 10),
    (MODEL_CPG, [768], (BC_SLIPWALL, BC_DIRICHLET), 10),
    (MODEL_CPG, [1023] * 20, (BC_PERIODIC, BC_PERIODIC), 4),      # the largest of many
    (MODEL_ONESTEP, [704] * 30, (BC_SLIPWALL, BC_DIRICHLET), 4),
    (MODEL_CPG, [63] * 700, (BC_ZEROGRAD, BC_DIRICHLET), 6),      # two groups of waves
    (MODEL_ONESTEP, [64] * 1100, (BC_SLIPWALL, BC_SLIPWALL), 6),
    (MODEL_ONESTEP, [20, 9, 17] * 1700, (BC_PERIODIC, BC_PERIODIC), 1030),   # two turns, two launches
    (MODEL_CPG, [300, 290] * 400, (BC_SLIPWALL, BC_ZEROGRAD), 6),
    (MODEL_ONESTEP, [600] * 520, (BC_ZEROGRAD, BC_DIRICHLET), 4),
    (MODEL_CPG, [40] * 600 + [700], (BC_ZEROGRAD, BC_DIRICHLET), 6),   # unlike: a launch for each capacity
    (MODEL_ONESTEP, [40, 700, 200, 300] * 150 + [3], (BC_SLIPWALL, BC_DIRICHLET), 700),
    (MODEL_CPG, [40] * 200 + [700], (BC_ZEROGRAD, BC_DIRICHLET), 6),   # all at once
])
def test_runs_equal_stage_launches(model, sizes, bc, nsteps):
    case = domains(model, sizes, bc)
    case.name = f"{len(sizes)} tiny domains"
    for a, b in zip(run(case, 0, nsteps), run(case, janc.PLAN_PER_LEVEL, nsteps)):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("noalloc", [False, True])
def test_dt_log_of_several_launches(noalloc):
    c = domains(MODEL_ONESTEP, [9], (BC_SLIPWALL, BC_SLIPWALL))
    torch, dev = torch_dev()
    ctx = janc.Context(c.model)
    D = c.domains[0]
    grid, phys = janc.make_grid(9, 1, D.dx, D.dy, D.bc, D.bc_prim), janc.physics_of(D)
    step = ctx.step_noalloc if noalloc else ctx.step
    out = []
    for parts in ([4200], [1400] * 3):   # 2048 steps a launch
        print(f"[gpu] {parts} steps of 9 cells, noalloc={noalloc}", flush=True)
        U, T = ctx.init_state(phys, torch.tensor(c.W.reshape(5, 1, 9), dtype=torch.float64, device=dev))
        t = torch.zeros(1, dtype=torch.float64, device=dev)
        logs = []
        for n in parts:
            logs.append(torch.zeros(n, dtype=torch.float64, device=dev))
            step(grid, phys, janc.make_time(cfl=0.4), U, T, n, t, logs[-1])
        ctx.sync_status()
        out.append([x.cpu().numpy() for x in (torch.cat(logs), U, T, t)])
    ctx.close()
    assert np.all(out[0][0] > 0.0)
    for a, b in zip(*out):
        assert np.array_equal(a, b)
