"""A tuned context computes the full operator on some of the blocks with a mapping of its own: every
selection matches the oracle after tuning, with the mapping set by hand, and untuned, on
lattices on both sides of the line between the split and the register-blocked kernel."""
import numpy as np
import pytest

import synth
from oracle import dirac, lattice

pytestmark = pytest.mark.gpu

TOL = {"f64": 8e-13, "f32": 1.6e-5}


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


# slices of 864 (ragged eighths) and 1120 sites, sites times rhs 8.3e4, 1.38e5 and 4.5e4, 1.8e5
@pytest.mark.parametrize("L,l0,nrhs", [((16, 12, 12, 12), 4, 3), ((16, 12, 12, 12), 4, 5), ((20, 10, 14, 16), 2, 1),
                                       ((20, 10, 14, 16), 2, 4)])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_parts_after_tuning(gu, L, l0, nrhs, prec):
    import paper_0710_0066_amd as sap
    print(f"parts L={L} nrhs={nrhs} {prec}", flush=True)
    k, P = 0.15, sap.SAP_F64 if prec == "f64" else sap.SAP_F32
    U = synth.gauge_field(L, 0.5, 1901)
    psi = synth.gaussian_spinor(L, 2901, nrhs=nrhs)
    ctx = gu.make_ctx(L, l0, k, U, max_rhs=nrhs)
    fin, fout = gu.to_sap(ctx, psi, nrhs, P), ctx.new_field(nrhs, P)
    W = dirac.apply_W(U, psi, k, l0)
    every = np.ones_like(lattice.site_mask(L, lattice.parity(L) >= 0))
    parts = [(sap.SAP_ALL, -1, every),
             (sap.SAP_BLACK, -1, lattice.site_mask(L, lattice.colour_x0_mask(L, l0, "black"))),
             (sap.SAP_WHITE, -1, lattice.site_mask(L, lattice.colour_x0_mask(L, l0, "white"))),
             (sap.SAP_ALL, 1, lattice.site_mask(L, lattice.single_block_mask(L, l0, 1)))]

    def check():
        for color, block, mask in parts:
            fout.fill_(3.0)
            sap.apply_W1_block(ctx, fout, fin, nrhs, 1, block, color, P)
            got = gu.from_sap(ctx, fout, nrhs, psi.shape, P)
            assert np.max(np.abs(got - W * mask)) <= TOL[prec] * np.max(np.abs(psi))
            assert np.all(got[np.broadcast_to(~mask.astype(bool), got.shape)] == 0)
        sap.apply_M(ctx, fout, fin, nrhs, P)
        got = gu.from_sap(ctx, fout, nrhs, psi.shape, P)
        assert np.max(np.abs(got - dirac.apply_M(U, psi, k))) <= TOL[prec] * np.max(np.abs(psi))

    check()
    sap.sap_tune(ctx, nrhs)
    check()
    for hop_map in (0, 11):
        sap.sap_set_hop_map(ctx, 1, P, nrhs, hop_map)
        check()
    sap.sap_set_hop_map(ctx, 1, P, nrhs, -1)
    check()
