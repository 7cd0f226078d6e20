"""The specialised chemistry kernels leave out the terms that a mechanism's structure makes
zero; which ones depends on whether the last species (the one not transported) takes part in
a reaction. Against the generic kernels, bitwise, with a reacting species last, an inert one
last, and with irreversible and third-body reactions only."""

import copy

import numpy as np
import pytest

import paper_2504_13750_amd as janc
from cases import synthetic_mechanism
from cases.amr import detailed_front_case
from gpu_util import run_uniform

pytestmark = pytest.mark.gpu


def _permuted(case, order):
    """The case with its species in another order."""
    c, m = copy.copy(case), copy.deepcopy(case.mech)
    for name in ("comp", "M", "nasa"):
        setattr(m, name, np.ascontiguousarray(np.asarray(getattr(m, name))[order]))
    for name in ("nu_f", "nu_b", "tb"):
        setattr(m, name, np.ascontiguousarray(np.asarray(getattr(m, name))[:, order]))
    m.species = [case.mech.species[k] for k in order]
    Y = np.concatenate([case.W[4:], 1.0 - case.W[4:].sum(0, keepdims=True)])[order]
    c.W = np.concatenate([case.W[:4], Y[:-1]])
    c.mech = m
    return c


def _kept(case, keep):
    """The case with some of its reactions."""
    c, m = copy.copy(case), copy.deepcopy(case.mech)
    for name in ("A", "b", "Ea", "nu_f", "nu_b", "tb", "has_tb", "reversible"):
        setattr(m, name, np.ascontiguousarray(np.asarray(getattr(m, name))[keep]))
    c.mech = m
    return c


@pytest.mark.parametrize("form", ["reacting last", "inert last", "third bodies", "irreversible"])
def test_structural_zeros_left_out_bitwise(form):
    base = detailed_front_case(nx=36, ny=20, mech=synthetic_mechanism())
    ns = len(base.mech.species)
    tb = np.asarray(base.mech.has_tb) != 0
    if form == "reacting last":
        c = _permuted(base, list(range(1, ns)) + [0])
    elif form == "inert last":
        c = _permuted(base, list(range(ns)))
    elif form == "third bodies":
        assert tb.any()
        c = _kept(_permuted(base, list(range(1, ns)) + [0]), np.flatnonzero(tb))
    else:
        c = _kept(base, np.flatnonzero(~tb))
        c.mech.reversible = np.zeros_like(c.mech.reversible)
    out = []
    for mode in (janc.CHEM_GENERIC, janc.CHEM_SPECIALIZED):
        ctx = janc.Context(janc.DETAILED, c.mech)
        ctx.chem_kernel = mode
        print(f"[gpu] {form}: mode {mode}", flush=True)
        out.append(run_uniform(c, 4, ctx=ctx))
        ctx.close()
    assert np.all(np.isfinite(out[0][0]))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


def test_structural_zeros_left_out_bitwise_in_reverse():
    from cases.amr import detailed_adjoint_case
    from gpu_util import torch_dev
    from test_gpu_adjoint_detailed import _dt
    a = detailed_adjoint_case(nx=24, ny=12, nsteps=2, mech=synthetic_mechanism())
    dt = _dt(a["case"], a["cfl_dt"])
    c = _permuted(a["case"], list(range(1, len(a["case"].mech.species))) + [0])
    torch, dev = torch_dev()
    out = []
    for mode in (janc.CHEM_GENERIC, janc.CHEM_SPECIALIZED):
        ctx = janc.Context(janc.DETAILED, c.mech)
        ctx.chem_kernel = mode
        print(f"[gpu] adjoint, reacting species last: mode {mode}", flush=True)
        W0 = torch.tensor(c.W, dtype=torch.float64, device=dev)
        loss, gW, gth = ctx.adjoint(janc.grid_of(c), janc.physics_of(c), janc.make_time(0.0, dt, 0.0),
                                    W0, 2, 2, a["probe_cell"], a["probe_w"])
        ctx.sync_status()
        out.append((loss.item(), gW.cpu().numpy(), gth.cpu().numpy()))
        ctx.close()
    (La, Ga, ta), (Lb, Gb, tb) = out
    assert La == Lb and np.array_equal(Ga, Gb) and np.array_equal(ta, tb)
    assert np.all(np.isfinite(Gb)) and np.max(np.abs(Gb[4:])) > 0
