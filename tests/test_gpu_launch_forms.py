"""The forms in which a plan's steps are launched, bitwise equal on the refined hierarchies:
workgroup order, halo table or look-up in the kernel, launches per level and per block, of the
synchronous and the crossover advance, with Lie and Strang splitting; and a second run of the
same call.
"""

import numpy as np
import pytest

import paper_2504_13750_amd as janc
from gpu_util import context_for, init_blocks, torch_dev
from test_gpu_blocks import _small_amr, _small_detailed_amr

pytestmark = pytest.mark.gpu


def run(bc, flags, width, linear, split, nsteps=3):
    print(f"[gpu] {bc.name} flags={flags} width={width} linear={linear} split={split}", flush=True)
    torch, dev = torch_dev()
    ctx = context_for(bc)
    plan = ctx.plan(janc.domains_of(bc), bc.blocks, bc.pool_cells, flags)
    plan.set_schedule(width, linear)
    U, T = init_blocks(ctx, bc)
    t = torch.zeros(len(bc.domains), dtype=torch.float64, device=dev)
    ctx.step_blocks(plan, janc.time_of(bc, split=split), U, T, nsteps, t)
    ctx.sync_status()
    out = U.cpu().numpy(), T.cpu().numpy(), t.cpu().numpy()
    plan.close()
    ctx.close()
    return out


SYNC = [(0, 16, 0), (0, 16, 1), (0, 32, 1), (janc.PLAN_RESOLVE_HALOS, 16, 1), (janc.PLAN_PER_LEVEL, 16, 1),
        (janc.PLAN_PER_LEVEL | janc.PLAN_RESOLVE_HALOS, 32, 0), (janc.PLAN_PER_BLOCK, 16, 1),
        (janc.PLAN_PER_BLOCK | janc.PLAN_RESOLVE_HALOS, 64, 0)]
CROSS = [(janc.PLAN_CROSSOVER | f, w, lin) for f, w, lin in
         [(0, 16, 0), (0, 16, 1), (0, 64, 1), (janc.PLAN_RESOLVE_HALOS, 32, 1)]]


@pytest.mark.parametrize("forms", [SYNC, CROSS], ids=["synchronous", "crossover"])
@pytest.mark.parametrize("detailed,split", [(False, janc.SPLIT_LIE), (True, janc.SPLIT_LIE), (True, janc.SPLIT_STRANG)])
def test_forms_agree_bitwise(forms, detailed, split):
    bc = _small_detailed_amr() if detailed else _small_amr()
    ref = run(bc, *forms[0], split)
    for form in forms:
        for a, b in zip(run(bc, *form, split), ref):
            assert np.array_equal(a, b), form
