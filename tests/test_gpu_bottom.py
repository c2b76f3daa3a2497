"""The psi V-cycle's coarse levels in one workgroup against the same levels as grid launches, and
against the oracle.

The reference V-cycle is put together from the single-kernel entry points, which launch one
grid kernel for each colour pass, defect restriction, prolongation and coarsest solve, in the
precision of the context; the solver's own V-cycle runs every level from 16^3 on in one
workgroup.

Tolerances, relative to the largest correction.  FP32: about 40 passes and transfers on the
deepest path, each a 13-term sum that keeps 13 * 2 * 2^-24 = 1.6e-6 of its largest value, add
6.2e-5; a defect's rounding, 2^-24 of its terms, comes back through the operator's condition
number (below 450 with K = 4: 180 / (12 h^2) on 32^3 cells of a box of 2 against 5 K^2 / 12 and
the lowest mode) as 2.7e-5: 1e-4.  FP64: the coarsest solves are accepted at a residual of
1e-12, their condition number is below 100: 1e-10.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2501_13046_amd import grtmg as g
from gpu_helpers import N, T, dev

pytestmark = pytest.mark.gpu
RULES = [g.BC_PERIODIC, g.BC_ROBIN, g.BC_REFLECT, g.BC_EXTRAP, g.BC_ZERO]
NU = (1, 3)
# first level in one workgroup and coarsest: 16 to 4 (alone, below 32^3), 10 to 5 (two cells a
# lane in the coarsest solve), 12 to 3, 8 to 4
SIDES = [(16, 3), (32, 4), (20, 3), (24, 4), (8, 2)]


def halved(a):
    """Mean of the 8 children."""
    n = a.shape[0] // 2
    return a.reshape(n, 2, n, 2, n, 2).sum(dim=(1, 3, 5)) * 0.125


def grid_cycle(s, level, levels, r, c):
    n, vt = r.shape[0], r.dtype
    d = torch.zeros((n,) * 3, dtype=vt, device=dev())
    if level == levels - 1:
        s.kernel_op(g.OP_COARSE_PSI, level, 0, r, d, None, c)
        return d

    def smooth(d, sweeps):
        for p in range(2 * sweeps):
            out = torch.full_like(d, np.nan)
            s.kernel_op(g.OP_PASS_PSI, level, p & 1, d, out, r, c)
            d = out
        return d
    d = smooth(d, NU[0])
    rc = torch.full((n // 2,) * 3, np.nan, dtype=vt, device=dev())
    s.kernel_op(g.OP_DEFECT_RESTRICT_PSI, level, 0, d, rc, r, c)
    dc = grid_cycle(s, level + 1, levels, rc, halved(c).contiguous())
    s.kernel_op(g.OP_PROLONG_ADD, level, 1, dc, d)
    return smooth(d, NU[1])


@pytest.mark.parametrize("n,levels", SIDES)
@pytest.mark.parametrize("bc", RULES)
@pytest.mark.parametrize("precision", [g.PREC_FP32_IR, g.PREC_FP64])
@pytest.mark.parametrize("cubic", [False, True])
def test_one_workgroup_matches_grid_launches(n, levels, bc, precision, cubic):
    f32 = precision == g.PREC_FP32_IR
    vt = torch.float32 if f32 else torch.float64
    kw = dict(bc=bc, length=2.0, origin=(-0.9, -1.1, -1.0), puncture_pos=(0.03, 0.0, -0.02), K=4.0,
              nu_pre=NU[0], nu_post=NU[1], cubic_prolong=cubic)
    p, po = g.params(n, levels, precision=precision, **kw), oracle.params(n, levels, **kw)
    rho5, rho1 = (synth.uniform_random(60 + k, (n,) * 3, 0, 0.05) for k in (0, 1))
    u0 = synth.uniform_random(62, (n,) * 3, -0.05, 0.05)
    s = g.Solver(p, T(rho5), T(rho1))
    u = T(u0)
    H, _, c = s.residual_fields(u, None, want_M=False)
    ref = N(grid_cycle(s, 0, levels, (-H).to(vt), c.to(vt)))
    s.vcycle(g.EQ_PSI, u, None)
    d = N(u) - u0
    uo, z3 = u0.copy(), np.zeros((3, n, n, n))
    oracle.step(po, 1, uo, z3.copy(), rho5, rho1, z3)
    size = np.abs(uo - u0).max()
    e_grid, e_orc = np.abs(d - ref).max() / size, np.abs(d - (uo - u0)).max() / size
    print(f"n={n} bc={bc} f32={f32} cubic={cubic}: grid launches {e_grid:.1e}, oracle {e_orc:.1e}", flush=True)
    assert e_grid < (1e-4 if f32 else 1e-10)
    assert e_orc < (1e-4 if f32 else 1e-10)


@pytest.mark.parametrize("bc", RULES)
@pytest.mark.parametrize("n,levels", [(36, 3), (28, 3)])
def test_block_solve_under_every_rule(n, levels, bc):
    """Coarsest levels of 9^3 and 7^3 cells, a launch of their own, in a definite system."""
    kw = dict(bc=bc, length=2.0, origin=(-0.9, -1.1, -1.0), puncture_pos=(0.03, 0.0, -0.02), K=4.0,
              nu_pre=NU[0], nu_post=NU[1])
    p, po = g.params(n, levels, **kw), oracle.params(n, levels, **kw)
    rho5, rho1 = (synth.uniform_random(70 + k, (n,) * 3, 0, 0.05) for k in (0, 1))
    u0 = synth.uniform_random(72, (n,) * 3, -0.05, 0.05)
    s, u, uo, z3 = g.Solver(p, T(rho5), T(rho1)), T(u0), u0.copy(), np.zeros((3, n, n, n))
    s.vcycle(g.EQ_PSI, u, None)
    oracle.step(po, 1, uo, z3.copy(), rho5, rho1, z3)
    assert np.abs(N(u) - uo).max() / np.abs(uo - u0).max() < 1e-10
