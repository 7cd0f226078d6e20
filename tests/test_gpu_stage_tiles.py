"""GPU parity of the RK stage kernel where its split of the work changes: species counts
whose component count leaves 0, 1, 2 or 3 over after rounds of four, every tile width, and
grids one cell short of, equal to and one cell beyond whole tiles and runs.

Bar: the repository's 1e-10 per conserved field (and T) against the oracle; tile widths
agree bitwise.
"""

import math

import numpy as np
import pytest

import oracle
import paper_2504_13750_amd as janc
from cases import (BlockCase, Case, Domain, MODEL_DETAILED, MODEL_ONESTEP, BC_DIRICHLET, BC_PERIODIC,
                   BC_SLIPWALL, BC_ZEROGRAD, detonation_tube_case, synthetic_mechanism)
from cases.common import make_blocks
from cases.mechanism import Mechanism
from gpu_util import rel_err, run_blocks, run_uniform

pytestmark = pytest.mark.gpu
TOL = 1e-10


def inert_mechanism(ns):
    """ns species with the seeded mechanism's thermodynamics (cyclically), no reactions."""
    m = synthetic_mechanism()
    pick = [k % m.ns for k in range(ns)]
    z = np.zeros((0, ns))
    return Mechanism(species=[f"S{k}" for k in range(ns)], elements=m.elements, comp=m.comp[pick],
                     M=m.M[pick] * (1.0 + 0.01 * np.arange(ns)), nasa=m.nasa[pick], A=np.zeros(0),
                     b=np.zeros(0), Ea=np.zeros(0), nu_f=z.astype(np.int32), nu_b=z.astype(np.int32),
                     tb=z, has_tb=np.zeros(0, np.int32), reversible=np.zeros(0, np.int32),
                     A_cgs=np.zeros(0), Ea_kcal=np.zeros(0))


def detailed_state(ns, nx, ny, bc, inflow=False):
    mech = inert_mechanism(ns)
    dx = 2e-5
    x, y = (np.arange(nx) + 0.5) / nx, (np.arange(ny) + 0.5) / ny
    X, Y = np.meshgrid(x, y)
    W = np.zeros((ns + 3, ny, nx))
    W[0] = 101325.0 * (2.0 + np.tanh(12.0 * (0.45 - X)) + 0.2 * np.sin(2 * math.pi * Y))
    W[1] = 80.0 + 30.0 * np.sin(2 * math.pi * X)
    W[2] = 40.0 * np.cos(2 * math.pi * (X + Y))
    W[3] = 900.0 + 500.0 * np.exp(-20.0 * (X - 0.5) ** 2)
    for k in range(ns - 1):
        W[4 + k] = (0.6 / ns) * (1.0 + 0.5 * np.sin(2 * math.pi * (X * (1 + k % 3) + 0.3 * k + Y)))
    prim = W[:, 0, -1].copy()
    return Case(name=f"mix{ns}_{nx}x{ny}", model=MODEL_DETAILED, nx=nx, ny=ny, dx=dx, dy=dx, bc=bc, W=W,
                mech=mech, cfl=0.4, bc_prim=[None, prim if inflow else None, None, None])


def check(case, nsteps):
    Ug, Tg, _, _ = run_uniform(case, nsteps)
    Uo, To = oracle.case_state(case)
    Uo, To, _, _, _ = oracle.step(case, Uo, To, nsteps)
    assert np.all(rel_err(Ug, Uo) <= TOL), rel_err(Ug, Uo)
    assert rel_err(Tg[None], To[None])[0] <= TOL


@pytest.mark.parametrize("ns", [2, 3, 4, 5, 7, 8, 11])
def test_species_counts_of_every_remainder(ns):
    check(detailed_state(ns, 37, 21, [BC_ZEROGRAD, BC_DIRICHLET, BC_SLIPWALL, BC_SLIPWALL], inflow=True), 3)


@pytest.mark.parametrize("nx,ny", [(15, 17), (16, 16), (17, 15), (3, 33), (65, 3), (31, 9), (255, 1), (256, 1),
                                   (257, 1), (5, 1)])
def test_tile_edges(nx, ny):
    bc = [BC_PERIODIC, BC_PERIODIC, BC_SLIPWALL, BC_ZEROGRAD]
    check(detailed_state(9, nx, ny, bc), 2)


def as_blocks(c):
    d = Domain(nx=c.nx, ny=c.ny, dx=c.dx, dy=c.dy, bc=c.bc, gamma=c.gamma, R=c.R, Q=c.Q, Ea=c.Ea, k=c.k,
               bc_prim=c.bc_prim)
    return BlockCase(name=c.name, model=c.model, domains=[d], blocks=make_blocks([(0, 0, 0, 0, c.nx, c.ny)]),
                     W=c.W.reshape(c.nU, -1), mech=c.mech, cfl=c.cfl)


@pytest.mark.parametrize("model,nx,ny", [(MODEL_ONESTEP, 129, 131), (MODEL_ONESTEP, 128, 128),
                                         (MODEL_DETAILED, 128, 128), (MODEL_DETAILED, 145, 128),
                                         (MODEL_ONESTEP, 16384, 1), (MODEL_ONESTEP, 16385, 1)])
def test_both_sides_of_the_quarter_tile_rule(model, nx, ny):
    """64 whole tiles are cut into quarters, 65 and more are not."""
    c = (detonation_tube_case(nx=nx, ny=ny) if model == MODEL_ONESTEP else
         detailed_state(9, nx, ny, [BC_ZEROGRAD, BC_DIRICHLET, BC_SLIPWALL, BC_SLIPWALL], inflow=True))
    check(c, 2)


@pytest.mark.parametrize("case", [
    detonation_tube_case(nx=70, ny=13), detonation_tube_case(nx=33, ny=35),
    detailed_state(6, 67, 11, [BC_ZEROGRAD, BC_DIRICHLET, BC_SLIPWALL, BC_SLIPWALL], inflow=True),
], ids=lambda c: c.name)
def test_tile_widths_agree_bitwise(case):
    bc = as_blocks(case)
    ref = run_blocks(bc, 3, tile=16)
    for tile, flags in [(32, 0), (64, 0), (16, janc.PLAN_RESOLVE_HALOS), (64, janc.PLAN_RESOLVE_HALOS)]:
        out = run_blocks(bc, 3, tile=tile, flags=flags)
        for a, b in zip(out, ref):
            assert np.array_equal(a, b), (tile, flags)
    if case.model == MODEL_ONESTEP:
        Uo, To = oracle.block_state(bc)
        Uo, To, _, _, _ = oracle.step_blocks(bc, Uo, To, 3)
        assert np.all(rel_err(ref[0], Uo) <= TOL)
