"""The entry of a call (T from U, first maxima) takes several tiles per workgroup in plans of
many tiles and publishes when the level or the domain changes. 820 copies of three uneven
domains, five tiles a copy (4100 tiles: domains change inside a workgroup's run, the last run
is full and runs start at every place of the pattern), bitwise equal to one copy alone."""

import numpy as np
import pytest

import paper_2504_13750_amd as janc
from cases import BlockCase, Domain, MODEL_CPG, MODEL_ONESTEP, BC_PERIODIC, BC_SLIPWALL, BC_ZEROGRAD
from cases.common import make_blocks
from gpu_util import init_blocks, torch_dev

pytestmark = pytest.mark.gpu

SIZES = [(8, 8), (20, 5), (16, 20)]
BCS = [[BC_PERIODIC] * 4, [BC_ZEROGRAD, BC_SLIPWALL, BC_SLIPWALL, BC_SLIPWALL], [BC_SLIPWALL] * 4]


def _case(model, copies):
    doms, recs, W = [], [], []
    for k in range(copies):
        rng = np.random.default_rng(11)
        for (nx, ny), bc in zip(SIZES, BCS):
            w = np.zeros((4 if model == MODEL_CPG else 5, nx * ny))
            w[0] = 1.0 + 0.3 * rng.uniform(-1, 1, nx * ny)
            w[1], w[2] = 0.2 * rng.uniform(-1, 1, (2, nx * ny))
            w[3] = (8.0 if model == MODEL_ONESTEP else 1.0) * (1.0 + 0.3 * rng.uniform(-1, 1, nx * ny))
            if model == MODEL_ONESTEP:
                w[4] = 0.7
            recs.append((len(doms), 0, 0, 0, nx, ny))
            doms.append(Domain(nx=nx, ny=ny, dx=0.01, dy=0.012, bc=bc, gamma=1.3, Q=20.0, Ea=8.0,
                               k=3.0 if model == MODEL_ONESTEP else 0.0, bc_prim=[None] * 4))
            W.append(w)
    return BlockCase(name=f"many{copies}", model=model, domains=doms, blocks=make_blocks(recs),
                     W=np.concatenate(W, axis=1), cfl=0.4)


def _run(bc, nsteps):
    print(f"[gpu] {bc.name} model={bc.model} nsteps={nsteps}", flush=True)
    torch, dev = torch_dev()
    ctx = janc.Context(bc.model)
    plan = ctx.plan(janc.domains_of(bc), bc.blocks, bc.pool_cells, 0)
    U, T = init_blocks(ctx, bc)
    t = torch.zeros(len(bc.domains), dtype=torch.float64, device=dev)
    ctx.step_blocks(plan, janc.make_time(cfl=0.4), U, T, nsteps, t)
    ctx.sync_status()
    out = U.cpu().numpy(), T.cpu().numpy(), t.cpu().numpy(), plan.stats()["tiles"]
    plan.close()
    ctx.close()
    return out


@pytest.mark.parametrize("model", [MODEL_CPG, MODEL_ONESTEP])
@pytest.mark.parametrize("nsteps", [1, 3])
def test_many_copies_equal_one(model, nsteps):
    copies = 820
    U1, T1, t1, n1 = _run(_case(model, 1), nsteps)
    U, T, t, n = _run(_case(model, copies), nsteps)
    assert n == copies * n1 and n >= 4096
    assert np.array_equal(U.reshape(U.shape[0], copies, -1), np.broadcast_to(U1[:, None], (U.shape[0], copies, U1.shape[1])))
    assert np.array_equal(T.reshape(copies, -1), np.broadcast_to(T1, (copies, T1.size)))
    assert np.array_equal(t.reshape(copies, -1), np.broadcast_to(t1, (copies, t1.size)))
