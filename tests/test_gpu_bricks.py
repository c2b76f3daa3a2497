"""psi kernels on LDS bricks (any even side and boundary rule), the pair kernels below
them and the marched W kernels of any even side, against the oracle: sides that are a multiple of the brick, that overhang it in y and
z, and that leave a half brick in x.

FP32 tolerances: a 13-term sum of weights that add up to 180 against a diagonal of 90 keeps
13 * 2 * 2^-24 = 1.6e-6 of the largest value; a restricted defect is such a sum itself (W: 135
taps whose weights add up to 300 against a diagonal of 100).
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2501_13046_amd import grtmg as g
from gpu_helpers import N, T, dev, rel_err

pytestmark = pytest.mark.gpu
RULES = [g.BC_PERIODIC, g.BC_ROBIN, g.BC_REFLECT, g.BC_EXTRAP, g.BC_ZERO]
SIDES = [(20, 3), (48, 4), (72, 4), (88, 4), (128, 6)]


def problem(n, levels, bc, precision):
    kw = dict(bc=bc, length=2.0, origin=(-0.9, -1.1, -1.0), puncture_pos=(0.03, 0.0, -0.02))
    return g.params(n, levels, precision=precision, **kw), oracle.params(n, levels, **kw)


def field(seed, n, lo, hi, f32):
    a = synth.uniform_random(seed, (n,) * 3, lo, hi)
    return a.astype(np.float32).astype(np.float64) if f32 else a


@pytest.mark.parametrize("n,levels", SIDES)
@pytest.mark.parametrize("bc", RULES)
@pytest.mark.parametrize("precision", [g.PREC_FP32_IR, g.PREC_FP64])
def test_pass_and_defect(n, levels, bc, precision):
    f32 = precision == g.PREC_FP32_IR
    vt = torch.float32 if f32 else torch.float64
    p, po = problem(n, levels, bc, precision)
    z = T(np.zeros((n,) * 3))
    s = g.Solver(p, z, z)
    d, r, c = (field(10 + k, n, lo, hi, f32) for k, (lo, hi) in enumerate([(-1, 1), (-500, 500), (-60, 5)]))
    for colour in (0, 1):
        out = torch.full((n,) * 3, np.nan, dtype=vt, device=dev())
        s.kernel_op(g.OP_PASS_PSI, 0, colour, T(d, vt), out, T(r, vt), T(c, vt))
        assert rel_err(N(out), oracle.pass_psi(po, d, r, c, colour)) < (2e-6 if f32 else 1e-13), colour
    out = torch.full((n // 2,) * 3, np.nan, dtype=vt, device=dev())
    s.kernel_op(g.OP_DEFECT_RESTRICT_PSI, 0, 0, T(d, vt), out, T(r, vt), T(c, vt))
    ref = oracle.restrict(r - (oracle.apply_lap(po, d) + c * d))
    assert rel_err(N(out), ref) < (2e-6 if f32 else 1e-12)


@pytest.mark.parametrize("n,levels", SIDES[1:])
@pytest.mark.parametrize("bc", RULES)
def test_residual_without_w(n, levels, bc):
    """H, c and the norms of a psi-only context, with a forcing."""
    p, po = problem(n, levels, bc, g.PREC_FP32_IR)
    p.K = po.K = 1.3
    u, f = field(20, n, -0.05, 0.05, False), field(21, n, -1, 1, False)
    rho5, rho1 = field(22, n, 0, 1, False), field(23, n, 0, 1, False)
    s = g.Solver(p, T(rho5), T(rho1), None, T(f))
    H, _, c = s.residual_fields(T(u), None, want_M=False)
    z3 = np.zeros((3, n, n, n))
    Ho, _, co = oracle.residuals(po, u, z3, rho5, rho1, z3, f)
    assert rel_err(N(H), Ho) < 1e-12
    assert rel_err(N(c), co) < 1e-13
    got = s.residual_norm(T(u), None)
    np.testing.assert_allclose(got[[0, 2]], oracle.norms(Ho)[[0, 2]], rtol=1e-11)


@pytest.mark.parametrize("nc", [3, 5, 9, 12, 20])
@pytest.mark.parametrize("bc", RULES)
@pytest.mark.parametrize("ncomp", [1, 3])
def test_cubic_prolongation_of_any_side(nc, bc, ncomp):
    """Tiles of 16 and 8 coarse cells in z that overhang the level."""
    if ncomp == 3 and bc != g.BC_PERIODIC:
        pytest.skip("vector corrections are periodic")
    n = 2 * nc
    levels = 3 if nc == 20 else 2
    p, po = problem(n, levels, bc, g.PREC_FP64)
    p.flags |= g.FLAG_CUBIC_PROLONG
    z = T(np.zeros((n,) * 3))
    s = g.Solver(p, z, z)
    poc = oracle.params(nc, 1, bc=bc, length=2.0, origin=(-0.9, -1.1, -1.0), puncture_pos=(0.03, 0.0, -0.02))
    C = synth.uniform_random(31, (ncomp,) + (nc,) * 3)
    F = synth.uniform_random(32, (ncomp,) + (n,) * 3)
    out = T(F)
    s.kernel_op(g.OP_PROLONG_ADD, 0, ncomp, T(C), out)
    ref = np.stack([F[a] + oracle.interp_cubic(poc, np.ascontiguousarray(C[a])) for a in range(ncomp)])
    assert rel_err(N(out), ref) < 1e-13


@pytest.mark.parametrize("n,levels", [(40, 4), (48, 4), (56, 4), (80, 5), (112, 5)])
@pytest.mark.parametrize("precision", [g.PREC_FP32_IR, g.PREC_FP64])
def test_ragged_w_columns(n, levels, precision):
    """The marched W pass, defect restriction and residual on sides that are no multiple of
    their rows: columns that overhang the grid, and a last column of fewer planes."""
    f32 = precision == g.PREC_FP32_IR
    vt = torch.float32 if f32 else torch.float64
    K = 1.7
    p = g.params(n, levels, K=K, precision=precision, solve_momentum=True)
    po = oracle.params(n, levels, K=K, solve_momentum=True)
    rho5, rho1 = field(40, n, 0, 1, False), field(41, n, 0, 1, False)
    S = synth.uniform_random(42, (3, n, n, n))
    s = g.Solver(p, T(rho5), T(rho1), T(S))
    d, r = synth.uniform_random(43, (3, n, n, n)), synth.uniform_random(44, (3, n, n, n), -500, 500)
    if f32:
        d, r = (a.astype(np.float32).astype(np.float64) for a in (d, r))
    for colour in (0, 1):
        out = torch.full((3, n, n, n), np.nan, dtype=vt, device=dev())
        s.kernel_op(g.OP_PASS_W, 0, colour, T(d, vt), out, T(r, vt))
        assert rel_err(N(out), oracle.pass_W(po, d, r, colour)) < (4e-6 if f32 else 1e-12), colour
    out = torch.full((3,) + (n // 2,) * 3, np.nan, dtype=vt, device=dev())
    s.kernel_op(g.OP_DEFECT_RESTRICT_W, 0, 0, T(d, vt), out, T(r, vt))
    defect = r - oracle.apply_deltaL(po, d)
    ref = np.stack([oracle.restrict(np.ascontiguousarray(defect[a])) for a in range(3)])
    assert rel_err(N(out), ref) < (1e-5 if f32 else 1e-12)
    u = field(45, n, -0.05, 0.05, False)
    W = synth.uniform_random(46, (3, n, n, n), -0.02, 0.02)
    H, M, c = s.residual_fields(T(u), T(W))
    Ho, Mo, co = oracle.residuals(po, u, W, rho5, rho1, S)
    assert rel_err(N(H), Ho) < 1e-12 and rel_err(N(M), Mo) < 1e-12 and rel_err(N(c), co) < 1e-13
    np.testing.assert_allclose(s.residual_norm(T(u), T(W)), oracle.norms(Ho, Mo), rtol=1e-11)


@pytest.mark.parametrize("n,levels", [(12, 2), (20, 3), (24, 4), (28, 3), (32, 4), (36, 3)])
@pytest.mark.parametrize("bc", RULES)
@pytest.mark.parametrize("cubic", [False, True])
def test_coarse_levels_in_one_workgroup(n, levels, bc, cubic):
    """One psi step in FP64 against the oracle's: coarsest levels of 3^3, 4^3, 5^3, 6^3, 7^3 and
    9^3 cells (one wave with one or two cells a lane, the block solve), first levels of the
    one-workgroup part from 6^3 to 16^3, both prolongations."""
    if n == 36 and bc == g.BC_REFLECT:
        pytest.skip("indefinite 9^3 system that the block BiCGSTAB does not solve to 1e-12 (singular flag)")
    kw = dict(bc=bc, length=2.0, origin=(-0.9, -1.1, -1.0), puncture_pos=(0.03, 0.0, -0.02), K=1.3,
              nu_pre=1, nu_post=3, cubic_prolong=cubic)
    p, po = g.params(n, levels, precision=g.PREC_FP64, **kw), oracle.params(n, levels, **kw)
    rho5, rho1 = field(60, n, 0, 0.05, False), field(61, n, 0, 0.05, False)
    s = g.Solver(p, T(rho5), T(rho1))
    uo = field(62, n, -0.05, 0.05, False)
    u = T(uo)
    z3 = np.zeros((3, n, n, n))
    for _ in range(2):
        s.vcycle(g.EQ_PSI, u, None)
        oracle.step(po, 1, uo, z3.copy(), rho5, rho1, z3)
    assert rel_err(N(u), uo) < 1e-11
