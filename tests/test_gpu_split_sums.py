"""The reductions that the split hop adds to its output, in solves: slots of the marching order on whole
and on ragged slices with some of the blocks selected, and more slots than the update kernels
add up themselves (above 4096 they are compressed first). A mapping without reductions (1 with
one right-hand side) runs the same hops and separate norm passes, and takes the same iterations."""
import numpy as np
import pytest
import torch

import synth
from oracle import dirac, lattice

pytestmark = pytest.mark.gpu

MARCH1, LANE4 = 11, 1


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


def options(sap, method, inner, tol):
    return sap.solve_opts(tol=tol, max_iter=2000, max_outer=20, inner_prec=sap.SAP_F32 if inner == "f32" else sap.SAP_F64,
                          inner_tol=1e-5 if inner == "f32" else 0.0,
                          method={"cg": sap.SAP_CG, "bicgstab": sap.SAP_BICGSTAB, "geom": sap.SAP_GEOM}[method])


@pytest.mark.parametrize("L,l0", [((4, 10, 14, 16), 2),       # 17.5 chunks of 64 sites per slice
                                  ((8, 8, 16, 16), 4)])       # 16 whole chunks per slice
@pytest.mark.parametrize("select", ["black", "block 1"])
@pytest.mark.parametrize("method", ["cg", "bicgstab", "geom"])
@pytest.mark.parametrize("inner", ["f32", "f64"])
def test_marching_slots_on_selected_blocks(gu, L, l0, select, method, inner):
    import paper_0710_0066_amd as sap
    print(f"marching slots L={L} {select} {method} {inner}", flush=True)
    k, tol = 0.11, 1e-10
    U = synth.gauge_field(L, 0.5, 1801)
    b = synth.gaussian_spinor(L, 2801)
    blk = 1 if select == "block 1" else -1
    mask = lattice.site_mask(L, lattice.single_block_mask(L, l0, 1) if blk == 1 else lattice.colour_x0_mask(L, l0, "black"))
    ctx = gu.make_ctx(L, l0, k, U)
    fb, fx = gu.to_sap(ctx, b, 1), ctx.new_field(1)
    count = {}
    for hop_map in (MARCH1, LANE4):
        sap.sap_set_hop_map(ctx, 0, sap.SAP_F32 if inner == "f32" else sap.SAP_F64, 1, hop_map)
        fx.fill_(3.0)
        info = sap.solve_blocks(ctx, fx, fb, 1, 1, sap.SAP_ALL if blk == 1 else sap.SAP_BLACK,
                                options(sap, method, inner, tol), block=blk)
        x = gu.from_sap(ctx, fx, 1, b.shape)
        assert np.all(x[~np.broadcast_to(mask, x.shape)] == 0)
        r = (b - dirac.apply_W(U, x, k, l0)) * mask
        assert np.linalg.norm(r) <= tol * np.linalg.norm(b * mask)
        count[hop_map] = [(e.iters, e.outer) for e in info]
    assert count[MARCH1] == count[LANE4]


@pytest.mark.parametrize("inner", ["f32", "f64"])
def test_more_than_4096_slots(gu, inner):
    import paper_0710_0066_amd as sap
    L, k, tol = (48, 24, 24, 24), 0.06, 1e-10          # 48 x 108 slots
    prec = sap.SAP_F32 if inner == "f32" else sap.SAP_F64
    U = synth.gauge_field(L, 0.35, 1802)
    b = synth.gaussian_spinor(L, 2802)
    ctx = gu.make_ctx(L, 4, k, U)
    fb, fx, first = gu.to_sap(ctx, b, 1), ctx.new_field(1), None
    for method in ("cg", "bicgstab", "geom"):
        count = {}
        for hop_map in (-1, LANE4):
            print(f"many slots {inner} {method} map {hop_map}", flush=True)
            sap.sap_set_hop_map(ctx, 0, prec, 1, hop_map)
            info = sap.solve_full(ctx, fx, fb, 1, options(sap, method, inner, tol))
            count[hop_map] = (info[0].iters, info[0].outer)
            if first is None:
                first = fx.clone()
                x = gu.from_sap(ctx, fx, 1, b.shape)
                assert np.linalg.norm(b - dirac.apply_M(U, x, k)) <= tol * np.linalg.norm(b)
            # |M^-1| <= 1 / (1 - 8 k): two solutions to tol differ by at most 4 tol |b|
            assert float((fx - first).norm()) <= 4 * tol * float(fb.norm())
        assert count[-1] == count[LANE4]
