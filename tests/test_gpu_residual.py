"""The outer loop of solve_full and solve_blocks: x_o = b_o + kappa D_oe x_e in FP64 leaves a
residual on the even sites only, whatever the precision and the method of the corrections, and
solves that need no correction, or cannot start one, answer without it."""
import numpy as np
import pytest

import synth
from oracle import dirac, lattice

pytestmark = pytest.mark.gpu

# one FP64 hop: kappa times 8 hops of products of 3 links each, rounded here and in the oracle
ODD_TOL = 64 * 2.0 ** -52


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("color", ["full", "all", "black", "block 1"])
@pytest.mark.parametrize("inner", ["f64", "f32", "f16"])
@pytest.mark.parametrize("method", ["cg", "bicgstab", "geom"])
def test_residual_is_left_on_the_even_sites(gu, color, inner, method):
    import paper_0710_0066_amd as sap
    L, l0, k, n = (8, 4, 2, 6), 2, 0.11, 3
    print(f"residual {color} {inner} {method}", flush=True)
    U = synth.gauge_field(L, 0.5, 1301)
    b = synth.gaussian_spinor(L, 2301, nrhs=n)
    o = sap.solve_opts(tol=1e-9, max_iter=100000, max_outer=60,
                       inner_prec={"f64": sap.SAP_F64, "f32": sap.SAP_F32, "f16": sap.SAP_F16}[inner],
                       inner_tol=1e-2, method={"cg": sap.SAP_CG, "bicgstab": sap.SAP_BICGSTAB, "geom": sap.SAP_GEOM}[method])
    ctx = gu.make_ctx(L, l0, k, U, max_rhs=n)
    fb, fx = gu.to_sap(ctx, b, n), ctx.new_field(n)
    fx.fill_(3.0)
    lb, mask = None, np.ones_like(lattice.site_mask(L, lattice.parity(L) >= 0))
    if color == "full":
        info = sap.solve_full(ctx, fx, fb, n, o)
    else:
        lb, blk = l0, 1 if color == "block 1" else -1
        mask = lattice.site_mask(L, lattice.single_block_mask(L, lb, 1) if blk == 1
                                 else lattice.colour_x0_mask(L, lb, color))
        info = sap.solve_blocks(ctx, fx, fb, n, 1, sap.SAP_BLACK if color == "black" else sap.SAP_ALL, o, block=blk)
    x = gu.from_sap(ctx, fx, n, b.shape)
    assert np.all(x[~np.broadcast_to(mask, x.shape)] == 0)
    r = (b - dirac.apply_op(U, x, k, lb)) * mask
    odd = lattice.site_mask(L, lattice.parity(L) == 1)
    assert np.max(np.abs(r * odd)) <= ODD_TOL * (np.max(np.abs(x)) + np.max(np.abs(b)))
    ax = tuple(range(1, r.ndim))
    assert np.all(np.sum(np.abs(r) ** 2, axis=ax) <= 1e-18 * np.sum(np.abs(b * mask) ** 2, axis=ax))
    assert max(e.true_rel_res for e in info) <= 1e-9


@pytest.mark.parametrize("method", ["cg", "bicgstab", "geom"])
def test_solves_without_a_correction(gu, method):
    import paper_0710_0066_amd as sap
    L, k, n = (4, 4, 2, 4), 0.11, 2
    print(f"no correction {method}", flush=True)
    U = synth.gauge_field(L, 0.5, 1302)
    b = synth.gaussian_spinor(L, 2302, nrhs=n)
    b[1] = 0
    m = {"cg": sap.SAP_CG, "bicgstab": sap.SAP_BICGSTAB, "geom": sap.SAP_GEOM}[method]
    ctx = gu.make_ctx(L, 2, k, U, max_rhs=n)
    fx = ctx.new_field(n)

    def solve(rhs, **kw):
        fx.fill_(3.0)
        o = sap.solve_opts(**{**dict(tol=1e-9, max_iter=1000, max_outer=20, method=m), **kw})
        return sap.solve_full(ctx, fx, gu.to_sap(ctx, rhs, n), n, o)

    # one zero right-hand side beside another: zero, with the count of the batch's corrections
    info = solve(b)
    x = gu.from_sap(ctx, fx, n, b.shape)
    assert np.all(x[1] == 0) and np.any(x[0] != 0)
    assert info[1].iters == 0 and info[1].true_rel_res == 0 and info[1].outer == info[0].outer > 0
    # nothing to do
    info = solve(np.zeros_like(b))
    assert all(e.iters == 0 and e.outer == 0 for e in info)
    assert float(fx.abs().max()) == 0
    # a non-finite source: refused before any correction, x = 0
    bad = b.copy()
    bad[0, 1, 0, 1, 2, 0, 0] = np.nan
    with pytest.raises(sap.SapError) as e:
        solve(bad)
    assert e.value.code == sap.SAP_E_NONFINITE
    assert float(fx.abs().max()) == 0
    # x = 0 as a solution, or no correction allowed: refused before any work
    for kw in (dict(tol=1.0), dict(max_outer=0), dict(max_iter=0)):
        with pytest.raises(sap.SapError) as e:
            solve(b, **kw)
        assert e.value.code == sap.SAP_E_ARG
        assert float(fx.min()) == 3
