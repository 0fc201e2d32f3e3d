"""The split hop kernel (a site's eight hops on eight wavefronts) against the oracle where its
work division can go wrong: slices of whole and of ragged 64-site chunks in the linear and
the x0-marching order, the smallest lattice, systems shorter than a chunk, one and several
right-hand sides, every precision, full, block-restricted and half-hop forms."""
import numpy as np
import pytest

import synth
from oracle import dirac, lattice

pytestmark = pytest.mark.gpu

F64_TOL, F32_TOL = 1e-13, 2e-6
# FP16 storage, of max |psi|: projection, link and output roundings of eight hops of a field
# of that size (the bounds of the FP16 operator tests)
F16_M_TOL, F16_HOP_TOL = 16 * 2.0 ** -12, 100 * 2.0 ** -12


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("L,l0", [((4, 2, 2, 2), 2),            # 8 sites per block and parity
                                  ((4, 10, 14, 16), 2),         # 17.5 chunks per slice: marching, ragged
                                  ((8, 8, 16, 16), 4),          # 16 whole chunks per slice: marching
                                  ((12, 6, 10, 12), 3)])        # linear, ragged blocks
@pytest.mark.parametrize("hop_map", [-1, 0, 11])
def test_split_hop_matches_oracle(gu, L, l0, hop_map):
    import paper_0710_0066_amd as sap
    print(f"split hop L={L} map {hop_map}", flush=True)
    k = 0.15
    U = synth.gauge_field(L, 0.5, 1201)
    par = lattice.parity(L)
    black = lattice.site_mask(L, lattice.colour_x0_mask(L, l0, "black"))
    for nrhs in (1, 3):
        psi = synth.gaussian_spinor(L, 2201, nrhs=nrhs)
        ctx = gu.make_ctx(L, l0, k, U, max_rhs=nrhs)
        big = float(np.max(np.abs(psi)))
        for prec, tol, hop_tol in ((sap.SAP_F64, F64_TOL * 8, F64_TOL * 8), (sap.SAP_F32, F32_TOL * 8, F32_TOL * 8),
                                   (sap.SAP_F16, F16_M_TOL, F16_HOP_TOL)):
            for full in (0, 1):
                sap.sap_set_hop_map(ctx, full, prec, nrhs, hop_map)
            fin, fout = gu.to_sap(ctx, psi, nrhs, prec), ctx.new_field(nrhs, prec)
            for parity in (0, 1):
                m_out = lattice.site_mask(L, par == parity)
                ref = dirac.hop(U, psi * lattice.site_mask(L, par != parity)) * m_out
                sap.apply_Dslash_eo(ctx, fout, fin, nrhs, parity, prec)
                got = gu.from_sap(ctx, fout, nrhs, psi.shape, prec) * m_out
                assert np.max(np.abs(got - ref)) <= hop_tol * big, (nrhs, prec, parity)
            sap.apply_M(ctx, fout, fin, nrhs, prec)
            got = gu.from_sap(ctx, fout, nrhs, psi.shape, prec)
            assert np.max(np.abs(got - dirac.apply_M(U, psi, k))) <= tol * big, (nrhs, prec)
            sap.apply_W1_block(ctx, fout, fin, nrhs, 1, -1, sap.SAP_BLACK, prec)
            got = gu.from_sap(ctx, fout, nrhs, psi.shape, prec)
            assert np.max(np.abs(got - dirac.apply_W(U, psi, k, l0) * black)) <= tol * big, (nrhs, prec)
            assert np.all(got[np.broadcast_to(~black, got.shape)] == 0)
